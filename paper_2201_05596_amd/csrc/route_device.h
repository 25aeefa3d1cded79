// Device-side pieces of the routing shared by the routing kernels and by the decode gate, which runs the whole
// routing at the end of its logits kernel (paper Sec. 5.4: top-k, the cumulative count that places a token inside
// its expert, the capacity cut and the mapping tables, fused into as few launches as the dependences allow).
#pragma once

#include "gate_common.h"

namespace moe {

// ------------------------------------------------------------------------------------------
// Top-k and gate weights of the tokens t0 .. t0 + n - 1 (n <= TB) by a block of NT threads, 16 lanes per token, and the
// chosen experts in e_sh [K][TB] (-1: no token).  NV > 0: rows of at most 16 NV logits, fetched for all rounds at once.
// ------------------------------------------------------------------------------------------
template <int K, int NV, int NT, int TB>
__device__ __forceinline__ void choose_experts(int32_t* e_sh, const float* __restrict__ logits, int t0, int n, int T, int E,
                                               int32_t* __restrict__ expert_idx, float* __restrict__ gate_w) {
    constexpr int PER = NT / 16, ROUNDS = (TB + PER - 1) / PER;
    static_assert(TB % PER == 0 || PER > TB, "whole rounds");
    const int tid = threadIdx.x, grp = tid >> 4, sub = tid & 15;
    auto publish = [&](int tl, Best g1, Best g2, float w1, float w2) {
        if (sub != 0 || tl >= TB) return;
        const bool ok = tl < n;
        e_sh[tl] = ok ? g1.i : -1;
        if (K == 2) e_sh[TB + tl] = ok ? g2.i : -1;
        if (ok) {
            const size_t o = (size_t)(t0 + tl) * K;
            expert_idx[o] = g1.i;
            gate_w[o] = w1;
            if (K == 2) {
                expert_idx[o + 1] = g2.i;
                gate_w[o + 1] = w2;
            }
        }
    };
    if (NV > 0) {
        constexpr int NVV = NV > 0 ? NV : 1;
        float v[ROUNDS][NVV];
        const int live_rounds = (n + PER - 1) / PER;                 // rounds that hold a token (uniform over the block)
#pragma unroll
        for (int it = 0; it < ROUNDS; ++it) {
            if (it >= live_rounds) break;
            const float* row = logits + (size_t)min(t0 + it * PER + grp, T - 1) * E;      // clamped: lanes stay in the moves
#pragma unroll
            for (int i = 0; i < NVV; ++i) v[it][i] = row[min(sub + 16 * i, E - 1)];
        }
#pragma unroll
        for (int it = 0; it < ROUNDS; ++it) {
            // no token in the round or in this wave (the waves share the vector ALUs): only the table entries
            if (it >= live_rounds || it * PER + __builtin_amdgcn_readfirstlane(grp) >= n) {
                publish(it * PER + grp, Best{}, Best{}, 0.f, 0.f);
                continue;
            }
#pragma unroll
            for (int i = 0; i < NVV; ++i) v[it][i] = sub + 16 * i < E ? v[it][i] : -INFINITY;
            Best g1, g2;
            float w1, w2;
            token_gate_regs<K, NVV>(v[it], E, sub, g1, g2, w1, w2);
            publish(it * PER + grp, g1, g2, w1, w2);
        }
    } else {
        for (int it = 0; it < ROUNDS; ++it) {
            Best g1, g2;
            float w1, w2;
            token_gate_mem<K>(logits + (size_t)min(t0 + it * PER + grp, T - 1) * E, E, sub, g1, g2, w1, w2);
            publish(it * PER + grp, g1, g2, w1, w2);
        }
    }
}

__host__ __device__ __forceinline__ int ceil_log2(int n) { return n > 1 ? 32 - __builtin_clz(n - 1) : 0; }

// f(expert, row) for the rows rows[e] .. C - 1 of every expert, each by one of the nthreads (a power of two, 64 at least): 2^sh
// adjacent threads per expert, so that no entry's number is divided by C.  All experts at once as long as that leaves eight threads each;
// fewer take a store of up to 64 lines per step, so beyond it is as many as the rows fill, up to a wave, and an expert after the
// other (us, all at once / so; top-1, 256 tokens, 256 rows per expert: 1024 experts 194 / 86, 512 88.8 / 46.0, 256 28.9 / 24.4; but 64
// tokens, 128 experts of 64 rows 4.2 / 4.8).
template <typename F>
__host__ __device__ __forceinline__ void for_unused_rows(const int32_t* rows, int E, int C, int tid, int nthreads, F f) {
    const int all = ceil_log2(nthreads) - ceil_log2(E), row = ceil_log2(C) < 6 ? ceil_log2(C) : 6, sh = all > 2 || all > row ? all : row;
    for (int e = tid >> sh; e < E; e += nthreads >> sh)
        for (uint32_t i = rows[e] + (tid & ((1 << sh) - 1)); i < (uint32_t)C; i += 1u << sh) f(e, i);     // C may be 2^31 - 1
}

// Launch order of the experts for the grouped GEMMs, which deal consecutive entries round-robin to
// the 8 XCDs.  Experts are ranked by kept rows (most first, ties by index); active ones are then
// handed out so that every XCD alternates between a busy expert (matrix-core bound) and a light one
// (weight-bandwidth bound), neighbouring XCDs in opposite phase: entry p = 8j + x (j-th expert of XCD
// x) takes the next busiest remaining expert when j + x is even, the next lightest when odd.  All
// XCDs get the same number of active experts, and while half of them multiply the others stream
// weights.  Experts without rows follow at the end.  O(active^2) compares, E <= 1024.
// order[E] (one entry past the list) holds twice the number of active experts plus a flag that
// tells the tiled GEMM how to deal its tiles to the XCDs: 1 when the active
// experts are of very different sizes (at least a quarter of them hold at most a quarter of the largest one's
// rows), so that dealing whole experts would leave the XCDs with unequal work; 0 otherwise.
// A second list follows at order[E + 1 ..]: the experts plainly by rows, busiest first, and the same entry at
// order[2E + 1] (for products whose tiles are long and few per compute unit: longest first, short ones fill the end).
// `order` holds 2E + 2 ints.  `sorted`, `active`: LDS scratch of E ints each; every thread of the block must call, at least E of
// them and a power of two; `rows` is visible to all.
// It ends the routing's chain on one compute unit, whose vector ALUs all its waves share, so what bounds it is the number of
// instructions: only active experts are ranked (one token has one or two), rows and index compared as one key, no scalar
// loops (an iteration is as long as an LDS round trip), no sums in LDS atomics, no exchanges between lanes through LDS.
// Decode gate of one token of 128 experts: 2.1 us of 9.0 before, 0.9 of 7.2 (16 tokens of 64: 1.5 of 10.3, 0.9 of 9.2).
__device__ __forceinline__ void write_expert_order(const int32_t* rows /* LDS */, int E, int32_t* __restrict__ order,
                                                   int32_t* sorted /* LDS */, int32_t* active /* LDS */, int tid, int nthreads) {
    // every wave counts the active experts by itself, and those before its own
    const int lane = tid % kWave, w = tid / kWave, bits = ceil_log2(E);
    const unsigned long long lt_mask = (1ull << lane) - 1;
    int na = 0, before = 0, r = 0;
    bool wide = false;                                          // keys of 32 bits hold rows below 2^20
    for (int g = 0; g * kWave < E; g += 2) {                    // two reads on their way at once
        const int e = g * kWave + lane;
        const int r0 = e < E ? rows[e] : 0, r1 = e + kWave < E ? rows[e + kWave] : 0;
        const unsigned long long m0 = __ballot(r0 > 0), m1 = __ballot(r1 > 0);
        if (w == g) { r = r0; before = na + __popcll(m0 & lt_mask); }
        na += __popcll(m0);
        if (w == g + 1) { r = r1; before = na + __popcll(m1 & lt_mask); }
        na += __popcll(m1);
        wide |= __ballot(max(r0, r1) >= 1 << 20) != 0;
    }
    if (tid < E) {
        if (r > 0) active[before] = wide ? tid : (r << bits) - tid;          // larger keys first, ties by index
        else sorted[na + tid - before] = tid;
    }
    __syncthreads();
    // rank of an active expert = number of active ones before it: 2^lp adjacent lanes (at most the 16 that exchange without
    // LDS) share an expert, each comparing it with a slice of the others
    const int lp = max(0, min(4, ceil_log2(nthreads) - ceil_log2(na)));
    const int slice = (na + (1 << lp) - 1) >> lp, lo = (tid & ((1 << lp) - 1)) * slice, hi = min(na, lo + slice), a = tid >> lp;
    if (na > 0 && a - (lane >> lp) < na) {                      // this wave has experts to rank
        const int mine = active[min(a, na - 1)];
        int rank = 0, e = mine;
        if (wide) {
            for (int o = lo; o < hi; ++o) {
                const int other = active[o], mr = rows[mine], ro = rows[other];
                rank += ro > mr || (ro == mr && other < mine) ? 1 : 0;
            }
        } else {
            e = -mine & ((1 << bits) - 1);
            int o = lo;
            for (; o + 8 <= hi; o += 8) {
                int k[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) k[i] = active[o + i];
#pragma unroll
                for (int i = 0; i < 8; ++i) rank += k[i] > mine ? 1 : 0;
            }
            for (; o < hi; ++o) rank += active[o] > mine ? 1 : 0;
        }
        if (lp > 0) rank += dpp_i<kDppSwap1>(rank);
        if (lp > 1) rank += dpp_i<kDppSwap2>(rank);
        if (lp > 2) rank += dpp_i<kDppHalfMirror>(rank);
        if (lp > 3) rank += dpp_i<kDppMirror>(rank);
        if (a < na && (tid & ((1 << lp) - 1)) == 0) sorted[rank] = e;
    }
    __syncthreads();
    // (a thread of the last wave, beside the first ones' look-ups) a quarter of the active experts hold at most a quarter of the
    // largest one's rows if the first of the last quarter does
    if (tid == nthreads - 1)
        order[E] = order[2 * E + 1] = 2 * na + (na > 0 && (long long)rows[sorted[na - (na + 3) / 4]] * 4 <= rows[sorted[0]] ? 1 : 0);
    if (tid < E) {
        const int p = tid, j = p >> 3, x = p & 7;
        // busy takes among positions 8j .. 8j+x-1: those x' with (j + x') even
        const int busy_before = 4 * j + ((j & 1) ? (x >> 1) : ((x + 1) >> 1));
        const int at = p >= na ? p : ((j + x) & 1) ? na - 1 - (p - busy_before) : busy_before;
        order[p] = sorted[at];
        order[E + 1 + p] = sorted[p];                     // second list: plainly by rows, busiest first
    }
}

// At most 256 tokens: the whole routing by one block of kSingleThreads threads, whose block-local ranks are already
// global ones; totals and ranks stay in LDS and registers, one memory round trip (the logits).  The block is as large as
// they come: the tokens' top-k is a chain of cross-lane moves, and four rounds of 64 tokens take a quarter of sixteen
// rounds of 16.  smem: route_single_lds_ints(E, K) ints.
constexpr int kSingleThreads = 1024;
template <int K, int NV>
__device__ __forceinline__ void route_single_body(int32_t* smem, const float* __restrict__ logits, int T, int E, int C,
                                                  int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot_idx,
                                                  float* __restrict__ gate_w, int32_t* __restrict__ expert_rows,
                                                  int32_t* __restrict__ slot_token, int32_t* __restrict__ expert_order) {
    constexpr int NW = kRouteTokens / kWave, NT = kSingleThreads;
    int32_t* e_sh = smem;                                       // [K][256] chosen expert per token
    int32_t* whist = smem + K * kRouteTokens;                   // [NW][K][E] tokens per (wave of tokens, choice, expert)
    int32_t* tot_sh = whist + NW * K * E;                       // [K][E] tokens per (choice, expert)
    int32_t* rows_sh = tot_sh + K * E;                          // [E]
    int32_t* sorted = rows_sh + E;                              // [E]
    const int tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
    for (int i = tid; i < NW * K * E; i += NT) whist[i] = 0;
    choose_experts<K, NV, NT, kRouteTokens>(e_sh, logits, 0, T, T, E, expert_idx, gate_w);
    __syncthreads();

    int my_e[K], my_rank[K];
    if (tid < kRouteTokens) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            my_e[j] = e_sh[j * kRouteTokens + tid];
            my_rank[j] = wave_rank_by_expert(my_e[j], lane, E, whist + (w * K + j) * E);
        }
    }
    __syncthreads();

    // prefix over the waves of tokens
    for (int i = tid; i < K * E; i += NT) {
        const int j = K == 2 && i >= E ? 1 : 0, e = i - j * E;
        int run = 0;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            const int c = whist[(ww * K + j) * E + e];
            whist[(ww * K + j) * E + e] = run;
            run += c;
        }
        tot_sh[i] = run;
    }
    __syncthreads();
    for (int e = tid; e < E; e += NT) {
        const int rows = min(tot_sh[e] + (K == 2 ? tot_sh[E + e] : 0), C);
        rows_sh[e] = rows;
        expert_rows[e] = rows;
    }
    if (tid < T) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int e = my_e[j];
            const int loc = my_rank[j] + whist[(w * K + j) * E + e] + (j == 1 ? tot_sh[e] : 0);   // second choices behind all first ones
            if (loc < C) slot_token[(size_t)e * C + loc] = tid;
            slot_idx[(size_t)tid * K + j] = loc < C ? loc : -1;
        }
    }
    __syncthreads();
    for_unused_rows(rows_sh, E, C, tid, NT, [&](int e, uint32_t i) { slot_token[(size_t)e * C + i] = -1; });
    if (expert_order) write_expert_order(rows_sh, E, expert_order, sorted, tot_sh, tid, NT);   // tot_sh: free by now
}
// LDS ints of route_single_body: chosen experts, per-wave histograms, totals, rows, order scratch
__host__ __device__ inline size_t route_single_lds_ints(int E, int k) {
    return (size_t)k * kRouteTokens + (size_t)(kRouteTokens / kWave) * k * E + (size_t)k * E + 2 * (size_t)E;
}

}  // namespace moe
