// Host side: a value for every call that no memory holds by accident.
#pragma once

#include <stdint.h>
#include <sys/random.h>
#include <time.h>
#include <unistd.h>

#include <atomic>

namespace moe {

// one-to-one on 64 bits, every bit of the result depends on every bit of z (finaliser of SplitMix64, Steele et al. 2014)
inline uint64_t mix64(uint64_t z) noexcept {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Never 0, never the same twice in a process (a counter through mix64), and 64 random bits to whoever does not know where
// this process began: what a scratch buffer happens to hold -- indices, counts, floats, another process' tags -- equals a
// call's tag with a probability of 2^-64 per word.  Safe from several threads; throws nothing.
inline uint64_t next_call_tag() noexcept {
    static const uint64_t first = []() noexcept {
        uint64_t v = 0;
        if (getrandom(&v, sizeof v, GRND_NONBLOCK) != (ssize_t)sizeof v) {
            timespec t{};
            clock_gettime(CLOCK_REALTIME, &t);
            v = mix64((uint64_t)t.tv_sec * 1000000000ull + (uint64_t)t.tv_nsec) ^ mix64((uint64_t)getpid());
        }
        return v;
    }();
    static std::atomic<uint64_t> calls{0};
    uint64_t tag;
    do tag = mix64(first + calls.fetch_add(1, std::memory_order_relaxed));
    while (tag == 0);
    return tag;
}

}  // namespace moe
