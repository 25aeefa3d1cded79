// Host side: what a kernel needs once on every device that it runs on.
#pragma once

#include <stdint.h>

#include <atomic>

namespace moe {

// A bit per device; past 64 of them nothing is remembered.  Safe from several threads: two that come first may both ask.
class OncePerDevice {
public:
    // ask() unless it has returned true on this device before
    template <typename F> bool operator()(int device, F ask) {
        const uint64_t bit = device >= 0 && device < 64 ? 1ull << device : 0;
        if (done_.load(std::memory_order_relaxed) & bit) return true;
        if (!ask()) return false;
        done_.fetch_or(bit, std::memory_order_relaxed);
        return true;
    }

private:
    std::atomic<uint64_t> done_{0};
};

}  // namespace moe
