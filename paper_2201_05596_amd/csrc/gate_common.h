// Per-token gate arithmetic shared by the routing kernels: top-k by logit with ties to the lowest
// expert index, softmax weight(s), computed by an aligned group of 16 lanes (paper Sec. 5.4: the
// gating function's top-k selection and its probability-domain weights).
#pragma once

#include "moe_internal.h"

namespace moe {

struct Best {
    float v;
    int i;
};
__device__ __forceinline__ Best better(Best a, Best b) {
    return (b.v > a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}
constexpr int kNoExpert = 0x7fffffff;
// later of a lane's experts against its best so far; a masked expert (-inf) is still one, so it beats none at all
__device__ __forceinline__ bool beats(float v, const Best& b) { return v > b.v || (v == b.v && b.i == kNoExpert); }
// All-reduce inside aligned groups of 16 lanes (one DPP "row") with data-parallel-primitive moves:
// swap inside pairs, swap pairs inside quads, mirror the two quads of each half row, mirror the two
// half rows.  After step i every aligned group of 2^i lanes holds one common value, which is what
// makes the mirrors (which reverse lane order) as good as butterflies.  No LDS traffic, unlike
// __shfl_xor.
constexpr int kDppSwap1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppSwap2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // row_half_mirror
constexpr int kDppMirror = 0x140;      // row_mirror
template <int CTRL> __device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}
template <int CTRL> __device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}
template <int CTRL> __device__ __forceinline__ Best best_step(Best a) {
    Best o;
    o.v = dpp_f<CTRL>(a.v);
    o.i = dpp_i<CTRL>(a.i);
    return better(a, o);
}
__device__ __forceinline__ Best group_best(Best a) {
    a = best_step<kDppSwap1>(a);
    a = best_step<kDppSwap2>(a);
    a = best_step<kDppHalfMirror>(a);
    a = best_step<kDppMirror>(a);
    return a;
}
// Sum in a fixed tree order; every lane ends with the same bits (each step adds the same two
// partial sums on both sides, and fp add commutes).
__device__ __forceinline__ float group_sum(float a) {
    a += dpp_f<kDppSwap1>(a);
    a += dpp_f<kDppSwap2>(a);
    a += dpp_f<kDppHalfMirror>(a);
    a += dpp_f<kDppMirror>(a);
    return a;
}

// exp on the hardware exp2 unit; the argument is <= 0 here and the dominant terms have a small
// argument, which keeps the softmax weights within ~1e-7 of the exact value
__device__ __forceinline__ float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

template <int K>
__device__ __forceinline__ void gate_weights(float s, Best g1, Best g2, float& w1, float& w2) {
    if (K == 1) {
        w1 = 1.0f / s;                          // softmax probability of the arg-max
        w2 = 0.f;
    } else {
        const float r = fast_exp(g2.v - g1.v);  // p2/p1; renormalised pair = (1, r)/(1 + r)
        w1 = 1.0f / (1.0f + r);
        w2 = r / (1.0f + r);
    }
}

// Top-K experts and gate weights of one token, computed by a group of 16 lanes; lane `sub` looks
// at experts sub, sub+16, ...  Every lane of the group returns the same result, experts below E whatever the logits are (NaN
// is no choice: a token with nothing else gets expert E - 1).
// Register version: the lane's NV logits are already loaded (padding = -inf).
template <int K, int NV>
__device__ __forceinline__ void token_gate_regs(const float (&v)[NV], int E, int sub, Best& g1, Best& g2, float& w1,
                                                float& w2) {
    const Best none{-INFINITY, kNoExpert};
    Best b1 = none, b2 = none;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int e = sub + 16 * i;
        if (beats(v[i], b1)) { b2 = b1; b1.v = v[i]; b1.i = e; }
        else if (beats(v[i], b2)) { b2.v = v[i]; b2.i = e; }
    }
    g1 = group_best(b1);
    g2 = none;
    if (K == 2) g2 = group_best(b1.i == g1.i ? b2 : b1);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) s += fast_exp(v[i] - g1.v);       // exp(-inf) = 0 for the padding
    gate_weights<K>(group_sum(s), g1, g2, w1, w2);
    g1.i = min(g1.i, E - 1);
    g2.i = min(g2.i, E - 1);
}
// Any E: two passes over the row in memory.
template <int K>
__device__ __forceinline__ void token_gate_mem(const float* __restrict__ row, int E, int sub, Best& g1, Best& g2,
                                               float& w1, float& w2) {
    const Best none{-INFINITY, kNoExpert};
    Best b1 = none, b2 = none;
    for (int e = sub; e < E; e += 16) {
        const float v = row[e];
        if (beats(v, b1)) { b2 = b1; b1.v = v; b1.i = e; }
        else if (beats(v, b2)) { b2.v = v; b2.i = e; }
    }
    g1 = group_best(b1);
    g2 = none;
    if (K == 2) g2 = group_best(b1.i == g1.i ? b2 : b1);
    float s = 0.f;
    for (int e = sub; e < E; e += 16) s += fast_exp(row[e] - g1.v);
    gate_weights<K>(group_sum(s), g1, g2, w1, w2);
    g1.i = min(g1.i, E - 1);
    g2.i = min(g2.i, E - 1);
}

// Rank of each lane's token among the wave's tokens that chose the same expert (e < 0: no token): the lanes with the
// same e are found bit by bit with ballots, whatever e is (E <= 2^bits); returns the number of lower ones; the lowest lane
// of every group of equal e writes the group's size to count[e] (LDS or global, one writer per expert and wave).
// One pass of `bits` ballots instead of one ballot and one lane exchange per distinct expert: 28 of those among 32 tokens
// of 128 experts.
__device__ __forceinline__ int wave_rank_by_expert(int e, int lane, int E, int32_t* count) {
    const unsigned long long lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    const int bits = 32 - __clz(E);                       // E >= 1; covers 0 .. E - 1
    unsigned long long same = __ballot(e >= 0);
    for (int b = 0; b < bits; b += 4) {                   // four ballots at a time; bits past the last are 0 in every e
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool one = e >> (b + i) & 1;
            const unsigned long long ones = __ballot(one);
            same &= one ? ones : ~ones;
        }
    }
    const int rank = __popcll(same & lt_mask);
    if (e >= 0 && rank == 0) count[e] = __popcll(same);
    return rank;
}

}  // namespace moe
