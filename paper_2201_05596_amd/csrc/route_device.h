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
            if (it >= live_rounds) {                                 // no token: only the table entries
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

// Launch order of the experts for the grouped GEMMs, which deal consecutive entries round-robin to
// the 8 XCDs.  Experts are ranked by kept rows (most first, ties by index); active ones are then
// handed out so that every XCD alternates between a busy expert (matrix-core bound) and a light one
// (weight-bandwidth bound), neighbouring XCDs in opposite phase: entry p = 8j + x (j-th expert of XCD
// x) takes the next busiest remaining expert when j + x is even, the next lightest when odd.  All
// XCDs get the same number of active experts, and while half of them multiply the others stream
// weights.  Experts without rows follow at the end.  O(E^2) compares, E <= 1024.
// order[E] (one entry past the list) tells the tiled GEMM how to deal its tiles to the XCDs: 1 when the active
// experts are of very different sizes (at least a quarter of them hold at most a quarter of the largest one's
// rows), so that dealing whole experts would leave the XCDs with unequal work; 0 otherwise.
// A second list follows at order[E + 1 ..]: the experts plainly by rows, busiest first, and the same flag at
// order[2E + 1] (for products whose tiles are long and few per compute unit: longest first, short ones fill the end).
// `order` holds 2E + 2 ints.  `sorted` is LDS scratch of E + 2 ints; every thread of the block must call.
__device__ __forceinline__ void write_expert_order(const int32_t* rows /* LDS */, int E, int32_t* __restrict__ order,
                                                   int32_t* sorted /* LDS */, int tid, int nthreads) {
    if (tid == 0) sorted[E] = sorted[E + 1] = 0;
    __syncthreads();
    // rank of expert e = number of experts that come before it.  With fewer experts than threads, `parts` adjacent
    // lanes share an expert, each comparing it with a slice of the others (8 independent LDS reads at a time).
    int parts = 1;
    while (parts < 16 && parts * 2 * E <= nthreads) parts *= 2;
    const int part = tid % parts, slice = (E + parts - 1) / parts;
    const int lo = part * slice, hi = min(E, lo + slice);
    int active = 0;
    for (int e0 = 0; e0 < E; e0 += nthreads / parts) {          // same trip count for every thread
        const int e = e0 + tid / parts;
        const bool ok = e < E;
        const int r = ok ? rows[e] : 0;
        int rank = 0, o = lo;
        for (; o + 8 <= hi; o += 8) {
            int ro[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) ro[i] = rows[o + i];
#pragma unroll
            for (int i = 0; i < 8; ++i) rank += (ro[i] > r || (ro[i] == r && o + i < e)) ? 1 : 0;
        }
        for (; o < hi; ++o) {
            const int ro = rows[o];
            rank += (ro > r || (ro == r && o < e)) ? 1 : 0;
        }
        for (int m = 1; m < parts; m <<= 1) rank += __shfl_xor(rank, m);
        if (ok && part == 0) {
            sorted[rank] = e;
            active += r > 0 ? 1 : 0;
        }
    }
    if (active) atomicAdd(&sorted[E], active);          // integer count in LDS: order-independent
    __syncthreads();
    const int na = sorted[E];
    {
        const int largest = rows[sorted[0]];
        int small = 0;
        for (int e = tid; e < E; e += nthreads) small += rows[e] > 0 && rows[e] * 4 <= largest ? 1 : 0;
        if (small) atomicAdd(&sorted[E + 1], small);
        __syncthreads();
        if (tid == 0) order[E] = order[2 * E + 1] = sorted[E + 1] * 4 >= na && na > 0 ? 1 : 0;
    }
    for (int p = tid; p < E; p += nthreads) {
        int e;
        if (p >= na) {
            e = sorted[p];
        } else {
            const int j = p >> 3, x = p & 7;
            // busy takes among positions 8j .. 8j+x-1: those x' with (j + x') even
            const int busy_before = 4 * j + ((j & 1) ? (x >> 1) : ((x + 1) >> 1));
            const int light_before = p - busy_before;
            e = ((j + x) & 1) ? sorted[na - 1 - light_before] : sorted[busy_before];
        }
        order[p] = e;
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
    int32_t* sorted = rows_sh + E;                              // [E + 2]
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
        const int j = i / E, e = i % E;
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
    for (uint32_t i = tid; i < (uint32_t)E * C; i += NT)        // E * C < 2^31
        if ((int)(i % (uint32_t)C) >= rows_sh[i / (uint32_t)C]) slot_token[i] = -1;
    if (expert_order) write_expert_order(rows_sh, E, expert_order, sorted, tid, NT);
}
// LDS ints of route_single_body: chosen experts, per-wave histograms, totals, rows, order scratch
__host__ __device__ inline size_t route_single_lds_ints(int E, int k) {
    return (size_t)k * kRouteTokens + (size_t)(kRouteTokens / kWave) * k * E + (size_t)k * E + 2 * (size_t)E + 2;
}

}  // namespace moe
