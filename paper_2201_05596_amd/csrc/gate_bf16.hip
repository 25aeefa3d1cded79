// Gate for bf16 tokens on the bf16 matrix cores, exact to fp32 level (paper Sec. 5.4: the gating
// function -- logits, top-k, the count that places a token inside its expert -- fused into as few
// kernels as the data dependences allow; it is small but sits on the critical path before every other
// kernel of the layer).
//
//   logits[t,e] = bg[e] + sum_i x[t,i] Wg[i,e],   x bf16, Wg and bg fp32, fp32 accumulation.
//
// An fp32 weight is the exact sum of three bf16 numbers (3 x 8 significant bits = the 24 of fp32):
// Wg = hi + mid + lo with hi = bf16(Wg), mid = bf16(Wg - hi), lo = bf16(Wg - hi - mid).  A bf16 token
// value times a bf16 piece is exact in fp32, so three v_mfma_f32_16x16x32_bf16 per tile give the same
// sum of exact products as an fp32 multiply-add chain, at a fraction of the fp32 matrix-core time.
//
// Kernels:
//   * gate_prepare_kernel writes the three pieces as ready-made MFMA B fragments (1 KB each: lane l
//     holds k = 8*(l/16)..+7 of expert column l%16), ordered [k-block][expert tile][piece]: once into a buffer the caller
//     keeps (packed gate weights), or into the workspace at every call of 2048 tokens or more; with fewer, kernels that
//     are given plain weights split them as they go;
//   * gate_bf16_kernel: a work-group owns a tile of 16*MA tokens x 16*NE experts; its four waves
//     split the k-blocks (wave w takes blocks w, w+4, ...) and each computes the whole tile for its
//     blocks, so no operand byte is fetched twice by a work-group.  Every operand fragment is one
//     16-byte load per lane from global memory straight into registers, several k-blocks ahead; no LDS
//     traffic and no barrier in the loop.  The four partial tiles are summed through LDS in a fixed
//     order, the finished tile is laid out [token][expert] in LDS and written with 16-byte stores.
//     When the tile spans all experts (K = 1 or 2) the kernel goes on to the first half of the
//     routing on the tile it holds: top-k and gate weights per token (16 lanes per token), the rank of
//     each token among the tile's tokens with the same expert (ballots) and the tile's histogram.
//     route_finalize_kernel turns ranks into rows.
//     With few tokens the experts are split over work-groups instead (K = 0: logits only) so that
//     more CUs take part, and the routing runs as a kernel of its own.
// Requires d_model to be a multiple of 32 and at most 128 experts; other shapes use the fp32 kernel.
#include "route_device.h"

namespace moe {

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

constexpr int kKB = 32;                  // k per MFMA
constexpr int kFragElems = 512;          // bf16 elements of one fragment (64 lanes x 8)
// KB k-blocks x ET expert tiles x 3 pieces; one thread per (k-block, expert tile, lane).
__global__ __launch_bounds__(256) void gate_prepare_kernel(const float* __restrict__ Wg, uint16_t* __restrict__ frags, int d,
                                                           int E, int KB, int ET) {
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)KB * ET * 64) return;
    const int lane = (int)(idx & 63);
    const long long fe = idx >> 6;
    const int et = (int)(fe % ET), kb = (int)(fe / ET);
    const int n = et * 16 + (lane & 15);
    const int k0 = kb * kKB + (lane >> 4) * 8;
    uint16_t p[3][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = k0 + j;
        const float w = (k < d && n < E) ? Wg[(size_t)k * E + n] : 0.f;
        const uint16_t hi = f32_to_bf16(w);
        const float r1 = w - bf16_to_f32(hi);                 // exact
        const uint16_t mid = f32_to_bf16(r1);
        const float r2 = r1 - bf16_to_f32(mid);               // exact
        p[0][j] = hi; p[1][j] = mid; p[2][j] = f32_to_bf16(r2);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        uint4 o;
        o.x = p[q][0] | ((uint32_t)p[q][1] << 16); o.y = p[q][2] | ((uint32_t)p[q][3] << 16);
        o.z = p[q][4] | ((uint32_t)p[q][5] << 16); o.w = p[q][6] | ((uint32_t)p[q][7] << 16);
        *reinterpret_cast<uint4*>(frags + ((size_t)(fe * 3 + q)) * kFragElems + lane * 8) = o;
    }
}

// Eight weights of one column (k = 8*(lane/16) .. +7) as gate_prepare_kernel splits them, for the kernels that read plain weights: a
// call of few tokens reads each weight so seldom that a launch for the split costs more than splitting as it goes (layers on plain
// weights, us: one token, 1024/4096, 128 experts 34.6 -> 27.8; 200 tokens of 32 112.6 -> 107.9; 2000 of 128 370 -> 362).
__device__ __forceinline__ void split_weights(const float (&v)[8], bf16x8_t (&piece)[3]) {
    float x[4][2];
    uint32_t u[3][4];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j / 2][j % 2] = v[j];
    split_bf16x3(x, u);
#pragma unroll
    for (int q = 0; q < 3; ++q) piece[q] = __builtin_bit_cast(bf16x8_t, make_uint4(u[q][0], u[q][1], u[q][2], u[q][3]));
}
// the weights themselves: column n of k-block kb, zero past E; Wg is [d, E]
__device__ __forceinline__ void load_weights(const float* __restrict__ Wg, int kb, int kg, int n, int E, float (&v)[8]) {
    const float* p = Wg + (size_t)(kb * kKB + kg * 8) * E + min(n, E - 1);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = p[(size_t)j * E];
}
__device__ __forceinline__ void zero_past(int n, int E, float (&v)[8]) {
    if (n >= E) {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = 0.f;
    }
}

template <int MA, int NE> struct GateCfg {
    static constexpr int PER = MA + 3 * NE;                                  // 16-byte loads per lane and k-block
    // k-blocks held in registers: as many as keep the CU's loads busy and divide the k-blocks of the usual widths (8 per wave with d =
    // 1024).  The last D of a wave fetch nothing; re-reading the last one instead, 3 to 6 deep, was up to half of all loads (8192
    // tokens, d = 1024, us: 32 experts 15.5 -> 9.4, 64 16.0 -> 13.4; 4001 tokens, top-2 of 32 13.6 -> 10.0; 777 tokens, logits
    // alone, 128 experts 7.6 -> 5.4; 128 experts stay at 20: 0.85 MB per CU at 50 GB/s).
    static constexpr int D = PER <= 16 ? 4 : 2;
};

// tile: MA token tiles (16 tokens each) x NE expert tiles; blockIdx.x = token tile, blockIdx.y = expert group;
// ET = expert tiles in all (fragment stride).  K = 0: logits only.  K = 1, 2 (needs NE == ET): also top-K, gate
// weights, tile-local ranks (parked in slot_idx) and histograms.
template <int MA, int NE, int K> struct GateLds {
    static constexpr int TM = 16 * MA, TN = 16 * NE;
    static constexpr int STRIDE = TN + 4;                         // floats per tile row: 4 rows apart fall 16 banks apart
    static constexpr int RED = 2 * MA * NE * 64 * 16;             // two partial tiles, bytes
    static constexpr int TILE = TM * STRIDE * 4;
    static constexpr int MAIN = RED > TILE ? RED : TILE;          // the finished tile reuses the partial tiles' space
    static constexpr int ROUTE = K > 0 ? (K * TM + K * TN) * 4 : 0;   // chosen experts, histogram
    static constexpr int BYTES = MAIN + ROUTE;
};

template <int MA, int NE, int K, bool PLAIN>
__device__ __forceinline__ void gate_bf16_body(char* lds, const uint16_t* __restrict__ x, const uint16_t* __restrict__ frags, const float* __restrict__ Wg,
                                               const float* __restrict__ bg, float* __restrict__ logits, int T, int d,
                                               int E, int ET, int32_t* __restrict__ expert_idx,
                                               int32_t* __restrict__ slot_idx, float* __restrict__ gate_w,
                                               int32_t* __restrict__ hist) {
    typedef GateLds<MA, NE, K> L;
    constexpr int D = GateCfg<MA, NE>::D, PER = GateCfg<MA, NE>::PER, WK = 4, TM = L::TM, TN = L::TN, STRIDE = L::STRIDE;
    f32x4_t* red = reinterpret_cast<f32x4_t*>(lds);               // [2][MA][NE][64]
    float* tile = reinterpret_cast<float*>(lds);                  // [TM][STRIDE], after the reduction

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wk = w;
    const int et0 = blockIdx.y * NE;                              // first expert tile of this work-group
    const int t0 = blockIdx.x * TM;
    const int KB = d / kKB;
    const int nkb = KB > wk ? (KB - wk + WK - 1) / WK : 0;        // k-blocks wk, wk + WK, ... of this wave

    // bias of this lane's expert columns, fetched before anything else is in flight
    float bias[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int col = (et0 + e) * 16 + (lane & 15);
        bias[e] = (bg && col < E) ? bg[col] : 0.f;
    }

    f32x4_t acc[MA][NE];
#pragma unroll
    for (int m = 0; m < MA; ++m)
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[m][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    if (nkb > 0) {
        // per-lane sources: token rows (clamped into the matrix: their results are never stored) and fragments
        const uint16_t* a_src[MA];
#pragma unroll
        for (int m = 0; m < MA; ++m)
            a_src[m] = x + (size_t)min(t0 + 16 * m + (lane & 15), T - 1) * d + (lane >> 4) * 8;
        const uint16_t* b_src = PLAIN ? nullptr : frags + (size_t)et0 * 3 * kFragElems + lane * 8;
        const size_t b_kb_stride = (size_t)ET * 3 * kFragElems;
        const int n0 = et0 * 16 + (lane & 15);                    // PLAIN: this lane's column of the first expert tile

        // Operands of one k-block: A fragments straight from the token rows, B fragments as stored.
        // Plain loads: the compiler tracks their completion.  (Loads issued from inline asm with
        // hand-placed waits are NOT an option here: the compiler regards an asm output as valid at once
        // and, under register pressure, copies it elsewhere before the data has arrived.)
        struct Stage {
            u32x4_t r[PLAIN ? MA : PER];                          // MA token fragments, then 3*NE weight fragments
            float wv[PLAIN ? NE : 1][8];                          // or the weights
        };
        auto load = [&](Stage& st, int step) {
            const int kb = wk + min(step, nkb - 1) * WK;          // past the end: harmless re-read, dropped
#pragma unroll
            for (int m = 0; m < MA; ++m) st.r[m] = *reinterpret_cast<const u32x4_t*>(a_src[m] + kb * kKB);
            if constexpr (PLAIN) {
#pragma unroll
                for (int e = 0; e < NE; ++e) load_weights(Wg, kb, lane >> 4, n0 + 16 * e, E, st.wv[e]);
            } else {
                const uint16_t* bp = b_src + (size_t)kb * b_kb_stride;
#pragma unroll
                for (int i = 0; i < 3 * NE; ++i) st.r[MA + i] = *reinterpret_cast<const u32x4_t*>(bp + i * kFragElems);
            }
        };
        auto mma = [&](Stage& st) {
            bf16x8_t af[MA], bf[NE][3];
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                if constexpr (PLAIN) {
                    zero_past(n0 + 16 * e, E, st.wv[e]);
                    split_weights(st.wv[e], bf[e]);
                } else {
#pragma unroll
                    for (int q = 0; q < 3; ++q) bf[e][q] = __builtin_bit_cast(bf16x8_t, st.r[MA + e * 3 + q]);
                }
            }
#pragma unroll
            for (int m = 0; m < MA; ++m) af[m] = __builtin_bit_cast(bf16x8_t, st.r[m]);
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int q = 0; q < 3; ++q)
#pragma unroll
                    for (int m = 0; m < MA; ++m)
                        acc[m][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[m], bf[e][q], acc[m][e], 0, 0, 0);
        };

        Stage st[D];
#pragma unroll
        for (int s = 0; s < D; ++s) load(st[s], s);
        int i = 0;
        for (; i + D < nkb; i += D) {                             // the last round fetches nothing
#pragma unroll
            for (int s = 0; s < D; ++s) {
                // the scheduling barriers pin "use the oldest, then fetch the block D ahead": left alone,
                // the compiler sinks the loads to their first use
                mma(st[s]);
                __builtin_amdgcn_sched_barrier(0);
                load(st[s], i + s + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < D; ++s)
            if (i + s < nkb) mma(st[s]);
    }

    // ---- sum of the four partial tiles, always as (w0 + w2) + (w1 + w3) ------------------------------
    if (w >= 2) {
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int e = 0; e < NE; ++e) red[(((w - 2) * MA + m) * NE + e) * 64 + lane] = acc[m][e];
    }
    __syncthreads();
    if (w < 2) {
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[m][e] += red[((w * MA + m) * NE + e) * 64 + lane];
    }
    __syncthreads();
    if (w == 1) {
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int e = 0; e < NE; ++e) red[(m * NE + e) * 64 + lane] = acc[m][e];
    }
    __syncthreads();
    if (w == 0) {
        // finished logits (bias added) go to LDS as [token][expert]; D fragment: column lane%16, rows 4*(lane/16)+r
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[m][e] += red[(m * NE + e) * 64 + lane];
        asm volatile("" ::: "memory");                                // keep the reads above ahead of the writes below
        // the partial tile just read and the finished tile share LDS: only this wave touches either here,
        // and its LDS operations execute in order
#pragma unroll
        for (int m = 0; m < MA; ++m)
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    tile[(16 * m + 4 * (lane >> 4) + r) * STRIDE + 16 * e + (lane & 15)] = acc[m][e][r] + bias[e];
    }
    __syncthreads();

    // ---- logits out: 16 bytes per thread, rows contiguous ------------------------------------------------
    {
        constexpr int V = TN / 4;                                 // float4 per tile row
        const int col0 = et0 * 16;
        for (int i = tid; i < TM * V; i += 256) {
            const int tl = i / V, c4 = (i % V) * 4;
            const int t = t0 + tl, col = col0 + c4;
            if (t >= T || col >= E) continue;
            const float4 v = *reinterpret_cast<const float4*>(tile + tl * STRIDE + c4);
            float* o = logits + (size_t)t * E + col;
            if ((E & 3) == 0) *reinterpret_cast<float4*>(o) = v;              // col + 3 < E and 16-byte aligned
            else {
                o[0] = v.x;
                if (col + 1 < E) o[1] = v.y;
                if (col + 2 < E) o[2] = v.z;
                if (col + 3 < E) o[3] = v.w;
            }
        }
    }

    if (K > 0) {
        constexpr int KK = K > 0 ? K : 1;
        int32_t* e_sh = reinterpret_cast<int32_t*>(lds + L::MAIN);    // [K][TM] chosen expert per token of the tile
        int32_t* h_sh = e_sh + KK * TM;                               // [K][TN] histogram of the tile
        for (int i = tid; i < KK * TN; i += 256) h_sh[i] = 0;
        // 16 lanes per token, 16 tokens at a time
        const int grp = tid >> 4, sub = tid & 15;
#pragma unroll
        for (int it = 0; it < MA; ++it) {
            const int tl = it * 16 + grp;
            float v[NE];
#pragma unroll
            for (int i = 0; i < NE; ++i) v[i] = sub + 16 * i < E ? tile[tl * STRIDE + sub + 16 * i] : -INFINITY;
            Best g1, g2;
            float w1, w2;
            token_gate_regs<KK, NE>(v, E, sub, g1, g2, w1, w2);
            if (sub == 0) {
                const int t = t0 + tl;
                const bool ok = t < T;
                e_sh[tl] = ok ? g1.i : -1;
                if (KK == 2) e_sh[TM + tl] = ok ? g2.i : -1;
                if (ok) {
                    expert_idx[(size_t)t * KK] = g1.i;
                    gate_w[(size_t)t * KK] = w1;
                    if (KK == 2) {
                        expert_idx[(size_t)t * KK + 1] = g2.i;
                        gate_w[(size_t)t * KK + 1] = w2;
                    }
                }
            }
        }
        __syncthreads();
        // one lane per token (the tile has at most 64): rank among the tile's tokens with the same expert
        if (w == 0) {
#pragma unroll
            for (int j = 0; j < KK; ++j) {
                const int e = lane < TM ? e_sh[j * TM + lane] : -1;
                const int rank = wave_rank_by_expert(e, lane, E, h_sh + j * TN);
                if (e >= 0) slot_idx[(size_t)(t0 + lane) * KK + j] = rank;
            }
        }
        __syncthreads();
        // histogram [K][E] of this tile
        for (int i = tid; i < KK * E; i += 256) {
            const int j = i / E, e = i % E;
            hist[(size_t)blockIdx.x * KK * E + i] = h_sh[j * TN + e];
        }
    }
}

template <int MA, int NE, int K, bool PLAIN>
__global__ __launch_bounds__(256) void gate_bf16_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ frags, const float* __restrict__ Wg,
                                                        const float* __restrict__ bg, float* __restrict__ logits, int T, int d,
                                                        int E, int ET, int32_t* __restrict__ expert_idx,
                                                        int32_t* __restrict__ slot_idx, float* __restrict__ gate_w,
                                                        int32_t* __restrict__ hist) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    gate_bf16_body<MA, NE, K, PLAIN>(lds, x, frags, Wg, bg, logits, T, d, E, ET, expert_idx, slot_idx, gate_w, hist);
}

// The whole gate of a decode step (at most 256 tokens) in ONE launch.  Bound by latencies: the gate weights' round trip,
// the hand-over, the chain of the routing.  A work-group of 16 waves computes the logits of 16 MA tokens for one tile of
// 16 experts, the waves sharing K between them, so that up to d = 2048 all operands are fetched in one round trip (four
// waves needed three); experts and tokens are split over work-groups so that many CUs share the read of the gate weights.
// Every work-group then publishes a flag, and the one with the highest index waits for all flags and runs the whole routing
// on the finished logits.  The flags lie in scratch memory that may hold anything, so a flag is the call's 64-bit tag: never
// 0, never repeated by the process, and not to be met by accident (next_call_tag; a small count of calls was, in memory that
// held indices or histograms before).  The waiting work-group puts every flag it has seen back to 0, which also makes a
// replayed graph launch (same tag) safe.
// Hand-over across the XCDs' separate L2s: logits and flags are written with device-scope stores (through the L2), a
// work-group waits for its logits stores to complete before it writes its flag, and the reader acquires at device scope
// (invalidate) before its loads.  The wait cannot hang: work-groups are started in index order, so all others are running or
// done when the last one starts (and the whole grid, at most 64 work-groups, fits on the chip at once); it is bounded all
// the same, and gives up (leaving wrong tables, never a hung GPU) after about 10^6 polls.
// One token, d = 1024, 128 experts: 12.4 us with four waves and a routing by 256 threads; 64 tokens, d = 2048: 23.2.
constexpr int kDecodeWaves = 16, kDecodeBlocks = 4;      // waves; k-blocks in flight per wave
template <int MA, int RK, int NV, bool PLAIN>
__global__ __launch_bounds__(kDecodeWaves * 64) void gate_decode_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ frags, const float* __restrict__ Wg, const float* __restrict__ bg, float* __restrict__ logits,
    int T, int d, int E, int ET, int C, int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot_idx,
    float* __restrict__ gate_w, int32_t* __restrict__ expert_rows, int32_t* __restrict__ slot_token,
    int32_t* __restrict__ expert_order, uint64_t* __restrict__ flags, uint64_t tag) {
    static_assert(kDecodeWaves * 64 == kSingleThreads, "the routing uses the same work-group");
    constexpr int TM = 16 * MA;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float* part = reinterpret_cast<float*>(lds);                 // [kDecodeWaves][TM][16]
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, kg = lane >> 4, et = blockIdx.y, t0 = blockIdx.x * TM;
    const int KB = d / kKB, nkb = KB > w ? (KB - w + kDecodeWaves - 1) / kDecodeWaves : 0;   // k-blocks w, w + 16, ...
    const int o_row = tid >> 4, o_col = et * 16 + (tid & 15);    // the logit that this thread finishes
    const float bias = bg && o_col < E ? bg[o_col] : 0.f;
    f32x4_t acc[MA];
#pragma unroll
    for (int m = 0; m < MA; ++m) acc[m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const uint16_t* a_src[MA];                                   // token rows, clamped: results past T are never stored
#pragma unroll
    for (int m = 0; m < MA; ++m) a_src[m] = x + (size_t)min(t0 + 16 * m + c, T - 1) * d + kg * 8;
    const uint16_t* b_src = PLAIN ? nullptr : frags + (size_t)et * 3 * kFragElems + lane * 8;
    for (int i0 = 0; i0 < nkb; i0 += kDecodeBlocks) {
        bf16x8_t a[kDecodeBlocks][MA], b[kDecodeBlocks][3];
        float wv[PLAIN ? kDecodeBlocks : 1][8];
#pragma unroll
        for (int i = 0; i < kDecodeBlocks; ++i) {
            if (i0 + i >= nkb) break;
            const int kb = w + (i0 + i) * kDecodeWaves;
#pragma unroll
            for (int m = 0; m < MA; ++m) a[i][m] = *reinterpret_cast<const bf16x8_t*>(a_src[m] + kb * kKB);
            if constexpr (PLAIN) {
                load_weights(Wg, kb, kg, et * 16 + c, E, wv[i]);
            } else {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    b[i][q] = *reinterpret_cast<const bf16x8_t*>(b_src + ((size_t)kb * ET * 3 + q) * kFragElems);
            }
        }
        __builtin_amdgcn_sched_barrier(0);                       // all loads go out before the first use
#pragma unroll
        for (int i = 0; i < kDecodeBlocks; ++i) {
            if (i0 + i >= nkb) break;
            if constexpr (PLAIN) {
                zero_past(et * 16 + c, E, wv[i]);
                split_weights(wv[i], b[i]);
            }
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int m = 0; m < MA; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][m], b[i][q], acc[m], 0, 0, 0);
        }
    }
#pragma unroll
    for (int m = 0; m < MA; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(w * TM + 16 * m + 4 * kg + r) * 16 + c] = acc[m][r];   // D: column lane % 16, rows 4 kg + r
    __syncthreads();
    if (o_row < TM && t0 + o_row < T && o_col < E) {
        float v = bias;
#pragma unroll
        for (int s = 0; s < kDecodeWaves; ++s) v += part[s * TM * 16 + tid];
        __hip_atomic_store(logits + (size_t)(t0 + o_row) * E + o_col, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int nblocks = gridDim.x * gridDim.y, bid = blockIdx.y * gridDim.x + blockIdx.x;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's logits have left the L2 ...
    __syncthreads();                                   // ... and every thread's of the work-group ...
    if (tid == 0) __hip_atomic_store(flags + bid, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ... before its flag
    if (bid != nblocks - 1) return;
    if (tid < nblocks) {
        int polls = 0;
        while (__hip_atomic_load(flags + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != tag && polls < (1 << 20)) {
            __builtin_amdgcn_s_sleep(1);
            ++polls;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); // nothing read below comes from a stale cache line
    // Each flag goes back to 0 (never a tag) once it has been seen: a captured launch that is replayed carries the
    // same tag every time and must not find it in the flags of its own previous run.
    if (tid < nblocks) __hip_atomic_store(flags + tid, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    route_single_body<RK, NV>(reinterpret_cast<int32_t*>(lds), logits, T, E, C, expert_idx, slot_idx, gate_w, expert_rows,
                              slot_token, expert_order);
}

template <int MA, int NE, int K, bool PLAIN>
int launch_cfg(const uint16_t* x, const uint16_t* frags, const float* Wg, const float* bg, float* logits, int T, int d, int E, int ET,
               int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* hist, hipStream_t s) {
    constexpr int smem = GateLds<MA, NE, K>::BYTES;
    static OncePerDevice asked;
    const int rc = ask_lds(reinterpret_cast<const void*>(&gate_bf16_kernel<MA, NE, K, PLAIN>), smem, asked);
    if (rc != MOE_OK) return rc;
    const dim3 grid((T + 16 * MA - 1) / (16 * MA), ET / NE);
    hipLaunchKernelGGL((gate_bf16_kernel<MA, NE, K, PLAIN>), grid, dim3(256), smem, s, x, frags, Wg, bg, logits, T, d, E, ET, expert_idx,
                       slot_idx, gate_w, hist);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// expert tiles, padded to 1, 2, 4 or 8
int padded_expert_tiles(int E) {
    const int et = (E + 15) / 16;
    return et <= 1 ? 1 : et <= 2 ? 2 : et <= 4 ? 4 : 8;
}

}  // namespace

bool gate_bf16_supported(int d, int E) { return d % kKB == 0 && d >= kKB && E >= 1 && E <= 128; }

size_t gate_bf16_ws_bytes(int d, int E) {
    if (!gate_bf16_supported(d, E)) return 0;
    return (size_t)(d / kKB) * padded_expert_tiles(E) * 3 * kFragElems * sizeof(uint16_t);
}

static int launch_prepare(const float* Wg, uint16_t* frags, int d, int E, int KB, int ET, hipStream_t s) {
    const long long threads = (long long)KB * ET * 64;
    hipLaunchKernelGGL(gate_prepare_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, Wg, frags, d, E, KB, ET);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

int launch_pack_gate(const float* Wg, void* packed, int d, int E, hipStream_t s) {
    if (!gate_bf16_supported(d, E)) return MOE_ERR_UNSUPPORTED;
    return launch_prepare(Wg, static_cast<uint16_t*>(packed), d, E, d / kKB, padded_expert_tiles(E), s);
}

// Wg_packed != nullptr: the gate weights as launch_pack_gate wrote them (Wg is then not used)
int launch_gate_logits_bf16(const void* x, const float* Wg, const void* Wg_packed, const float* bg, float* logits, int T,
                            int d, int E, hipStream_t s) {
    if (!gate_bf16_supported(d, E) || (!Wg && !Wg_packed)) return MOE_ERR_INVALID_ARG;
    const int ET = padded_expert_tiles(E);
    const uint16_t* frags = static_cast<const uint16_t*>(Wg_packed);
    const uint16_t* xb = static_cast<const uint16_t*>(x);
    // One expert tile: most work-groups, least time per CU.  64 tokens instead of 32 (fewer operand bytes per output) where that still
    // gives every CU a work-group; with the fewer than 2048 tokens that come here larger tiles never would.
    const int tokens = (long long)((T + 63) / 64) * ET >= 256 ? 64 : 32;
#define MOE_GATE_CASE(ma) \
    return frags ? launch_cfg<ma, 1, 0, false>(xb, frags, nullptr, bg, logits, T, d, E, ET, nullptr, nullptr, nullptr, nullptr, s) \
                 : launch_cfg<ma, 1, 0, true>(xb, nullptr, Wg, bg, logits, T, d, E, ET, nullptr, nullptr, nullptr, nullptr, s)
    if (tokens == 64) MOE_GATE_CASE(4);
    MOE_GATE_CASE(2);
#undef MOE_GATE_CASE
}

// The decode gate in one launch: bf16 tokens, at most 256 of them.  flags: kGateFlags words of scratch, whatever they hold;
// tag: next_call_tag().
bool gate_decode_supported(int T, int d, int E) { return gate_bf16_supported(d, E) && T <= kRouteTokens; }

template <int MA, int RK, int NV, bool PLAIN>
static int launch_decode_p(const uint16_t* x, const uint16_t* frags, const float* Wg, const float* bg, float* logits, int T, int d, int E,
                             int ET, int C, int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* expert_rows,
                             int32_t* slot_token, int32_t* expert_order, uint64_t* flags, uint64_t tag, hipStream_t s) {
    const size_t route = route_single_lds_ints(E, RK) * sizeof(int32_t), sums = (size_t)kDecodeWaves * 16 * MA * 16 * 4;
    const dim3 grid((T + 16 * MA - 1) / (16 * MA), ET);              // smallest tiles: most work-groups (at most 8 x 8)
    if (grid.x * grid.y > kGateFlags) return MOE_ERR_INVALID_ARG;
    hipLaunchKernelGGL((gate_decode_kernel<MA, RK, NV, PLAIN>), grid, dim3(kDecodeWaves * 64), route > sums ? route : sums, s, x, frags, Wg,
                       bg, logits, T, d, E, ET, C, expert_idx, slot_idx, gate_w, expert_rows, slot_token, expert_order, flags, tag);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

template <int MA, int RK, int NV>
static int launch_decode_cfg(const uint16_t* x, const uint16_t* frags, const float* Wg, const float* bg, float* logits, int T, int d, int E,
                             int ET, int C, int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* expert_rows,
                             int32_t* slot_token, int32_t* expert_order, uint64_t* flags, uint64_t tag, hipStream_t s) {
    return frags ? launch_decode_p<MA, RK, NV, false>(x, frags, nullptr, bg, logits, T, d, E, ET, C, expert_idx, slot_idx, gate_w, expert_rows,
                                                      slot_token, expert_order, flags, tag, s)
                 : launch_decode_p<MA, RK, NV, true>(x, nullptr, Wg, bg, logits, T, d, E, ET, C, expert_idx, slot_idx, gate_w, expert_rows,
                                                     slot_token, expert_order, flags, tag, s);
}

int launch_gate_decode(const void* x, const float* Wg, const void* Wg_packed, const float* bg, float* logits, int T, int d,
                       int E, int k, int C, int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* expert_rows,
                       int32_t* slot_token, int32_t* expert_order, uint64_t* flags, uint64_t tag, hipStream_t s) {
    if (!gate_decode_supported(T, d, E) || (!Wg && !Wg_packed) || !flags || k < 1 || k > 2) return MOE_ERR_INVALID_ARG;
    const int ET = padded_expert_tiles(E);
    const uint16_t* frags = static_cast<const uint16_t*>(Wg_packed);
    const uint16_t* xb = static_cast<const uint16_t*>(x);
#define MOE_DECODE_CASE(kk, nv) \
    return T <= 128 ? launch_decode_cfg<1, kk, nv>(xb, frags, Wg, bg, logits, T, d, E, ET, C, expert_idx, slot_idx, gate_w, \
                                                   expert_rows, slot_token, expert_order, flags, tag, s)              \
                    : launch_decode_cfg<2, kk, nv>(xb, frags, Wg, bg, logits, T, d, E, ET, C, expert_idx, slot_idx, gate_w, \
                                                   expert_rows, slot_token, expert_order, flags, tag, s)
    if (k == 1) {
        if (E <= 16) MOE_DECODE_CASE(1, 1);
        if (E <= 32) MOE_DECODE_CASE(1, 2);
        if (E <= 64) MOE_DECODE_CASE(1, 4);
        MOE_DECODE_CASE(1, 8);
    }
    if (E <= 16) MOE_DECODE_CASE(2, 1);
    if (E <= 32) MOE_DECODE_CASE(2, 2);
    if (E <= 64) MOE_DECODE_CASE(2, 4);
    MOE_DECODE_CASE(2, 8);
#undef MOE_DECODE_CASE
}

// With fewer tokens the fused kernel would leave most CUs idle; logits over expert groups plus a separate
// routing kernel is faster then.
bool gate_bf16_fused_supported(int T, int d, int E) { return gate_bf16_supported(d, E) && T >= 2048; }

int launch_gate_bf16_fused(const void* x, const float* Wg, const void* Wg_packed, const float* bg, float* logits, int T,
                           int d, int E, int k, int32_t* expert_idx, int32_t* slot_idx, float* gate_w, void* frag_ws,
                           int32_t* scratch, int* tokens_per_hist, const int32_t** hist_out, hipStream_t s) {
    if (!gate_bf16_fused_supported(T, d, E) || (!frag_ws && !Wg_packed) || !scratch || k < 1 || k > 2)
        return MOE_ERR_INVALID_ARG;
    const int KB = d / kKB, ET = padded_expert_tiles(E);
    const uint16_t* frags = static_cast<const uint16_t*>(Wg_packed);
    // 64-token tiles once they give every CU a work-group, else 32-token ones
    const int MA = (T + 63) / 64 >= 256 ? 4 : 2;
    const int TM = 16 * MA;
    int32_t* hist = scratch;                                      // one histogram per tile: route_scratch_ints(T, E, k)
    int rc = MOE_OK;
    if (!frags) {
        rc = launch_prepare(Wg, static_cast<uint16_t*>(frag_ws), d, E, KB, ET, s);
        if (rc != MOE_OK) return rc;
        frags = static_cast<const uint16_t*>(frag_ws);
    }
    const uint16_t* xb = static_cast<const uint16_t*>(x);
    rc = MOE_ERR_INVALID_ARG;
#define MOE_GATE_CASE(ma, ne, kk) \
    if (MA == ma && ET == ne && k == kk) \
    rc = launch_cfg<ma, ne, kk, false>(xb, frags, nullptr, bg, logits, T, d, E, ET, expert_idx, slot_idx, gate_w, hist, s)
    MOE_GATE_CASE(4, 8, 1); MOE_GATE_CASE(4, 4, 1); MOE_GATE_CASE(4, 2, 1); MOE_GATE_CASE(4, 1, 1);
    MOE_GATE_CASE(2, 8, 1); MOE_GATE_CASE(2, 4, 1); MOE_GATE_CASE(2, 2, 1); MOE_GATE_CASE(2, 1, 1);
    MOE_GATE_CASE(4, 8, 2); MOE_GATE_CASE(4, 4, 2); MOE_GATE_CASE(4, 2, 2); MOE_GATE_CASE(4, 1, 2);
    MOE_GATE_CASE(2, 8, 2); MOE_GATE_CASE(2, 4, 2); MOE_GATE_CASE(2, 2, 2); MOE_GATE_CASE(2, 1, 2);
#undef MOE_GATE_CASE
    *tokens_per_hist = TM;
    *hist_out = hist;
    return rc;
}

}  // namespace moe
