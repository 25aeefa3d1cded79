// Gating kernels for gfx950: gate logits, softmax + top-k, and the capacity
// prefix count that gives every (token, choice) its row inside its expert.
//
// Paper Sec. 5.4: the gating function is top-k, a cumulative sum that yields the
// position of each token among those processed by its expert (bounded by the
// capacity), and a scatter, all driven by a dense token-to-expert mapping table
// instead of one-hot masks.  The paper parallelises the cumsum with a Blelloch
// scan on its hardware; here the count is done with 64-wide wavefront ballots
// (rank inside a wave), a per-tile histogram and a prefix over tiles, which
// is deterministic (no atomics) and needs two small launches.
#include <type_traits>

#include "route_device.h"

namespace moe {

// ------------------------------------------------------------------------------------------
// logits[t,e] = bg[e] + sum_i x[t,i] Wg[i,e]     fp32 in, fp32 accumulate, on the fp32 matrix cores
//
// v_mfma_f32_16x16x4_f32: a wave owns 16 tokens x 64 experts (4 accumulator tiles).  Per 32-wide
// k-chunk a lane reads 8 consecutive k of its token row straight from global memory (16 bytes of
// bf16, widened by a shift, or 32 bytes of fp32) and feeds them to 8 successive MFMAs; lane group
// g = lane/16 therefore holds k = 8g + j in MFMA j, and reads the matching Wg row 8g + j from an
// LDS tile kept in Wg's own [k][e] layout (columns rotated by 16 per 8 rows so that the four lane
// groups hit different banks).  No transposition anywhere.  A work-group is WT x WE x WK waves:
// token tiles x 64-expert tiles x k-splits (the k-split, summed through LDS in fixed order, keeps
// every CU busy when there are few tokens).
// ------------------------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));
constexpr int kGK = 32;      // k-rows per step
constexpr int kGPD = 3;      // steps of operands kept in flight in registers
constexpr int kLogitsTokens = 16;   // tokens of a work-group that also routes them

// 8 consecutive k of a token row as raw 16-byte words (bf16: one word; fp32: two), widened later
template <typename XT> struct XRaw;
template <> struct XRaw<uint16_t> {
    uint4 w;
    __device__ __forceinline__ void load(const uint16_t* row, int k, int d) {
        w = *reinterpret_cast<const uint4*>(row + min(k, d - 8));
    }
    __device__ __forceinline__ void widen(int k, int d, float (&v)[8]) const {
        const bool in = k < d;                              // d % 8 == 0: all eight or none
        const uint4 a = in ? w : make_uint4(0, 0, 0, 0);
        v[0] = __uint_as_float(a.x << 16); v[1] = __uint_as_float(a.x & 0xffff0000u);
        v[2] = __uint_as_float(a.y << 16); v[3] = __uint_as_float(a.y & 0xffff0000u);
        v[4] = __uint_as_float(a.z << 16); v[5] = __uint_as_float(a.z & 0xffff0000u);
        v[6] = __uint_as_float(a.w << 16); v[7] = __uint_as_float(a.w & 0xffff0000u);
    }
};
template <> struct XRaw<float> {
    float4 lo, hi;
    __device__ __forceinline__ void load(const float* row, int k, int d) {
        lo = *reinterpret_cast<const float4*>(row + min(k, d - 4));
        hi = *reinterpret_cast<const float4*>(row + min(k + 4, d - 4));
    }
    __device__ __forceinline__ void widen(int k, int d, float (&v)[8]) const {
        const bool in0 = k < d, in1 = k + 4 < d;            // d % 4 == 0
        v[0] = in0 ? lo.x : 0.f; v[1] = in0 ? lo.y : 0.f; v[2] = in0 ? lo.z : 0.f; v[3] = in0 ? lo.w : 0.f;
        v[4] = in1 ? hi.x : 0.f; v[5] = in1 ? hi.y : 0.f; v[6] = in1 ? hi.z : 0.f; v[7] = in1 ? hi.w : 0.f;
    }
};

// VEC = 4: E is a multiple of 4 and Wg rows are read as float4; VEC = 1: any E, scalar reads.
// FULL: d is a multiple of 32*WK and E of the work-group's expert width, so no operand is ever out
// of range and the selects that zero them disappear from the loop.
// K > 0 (four k-splits, at most 64 experts): the kernel goes on to what route_tile_kernel does for its 16 tokens.  The logits of
// a token lie in 16 adjacent lanes as the top-k wants them, a wave finishes four tokens: about 1 us more than the logits alone
// where that kernel is a launch of 4.8.  moe_gate, fp32, two launches / one before the finalising kernel, us, captured in a graph: 1536
// tokens, d = 512, 8 experts, top-2 15.3 / 14.0; 2500, d = 2048, 8 experts 29.1 / 28.5; 4096, d = 2048, 64 experts 30.0 / 27.7.
template <typename XT, int WT, int WE, int WK, int VEC, bool FULL, int K = 0>
__global__ __launch_bounds__(256) void gate_logits_kernel(const XT* __restrict__ x, const float* __restrict__ Wg,
                                                          const float* __restrict__ bg, float* __restrict__ logits,
                                                          int T, int d, int E, int32_t* __restrict__ expert_idx = nullptr,
                                                          int32_t* __restrict__ slot_idx = nullptr, float* __restrict__ gate_w = nullptr,
                                                          int32_t* __restrict__ hist = nullptr) {
    static_assert(WT * WE * WK == 4, "four waves");
    static_assert(K == 0 || WK == 4, "a wave finishes a row of each group of four");
    constexpr int EN = WE * 64;                       // experts per pass of the work-group
    constexpr int TM = WT * 16;                       // tokens per work-group
    constexpr int NB = WK * kGK * EN / 256 / VEC;     // Wg words staged per thread and step
    __shared__ __attribute__((aligned(16))) float Bs[WK][kGK][EN];
    __shared__ float red[WK > 1 ? (WK - 1) * WT * WE * 16 * 64 : 1];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n = lane & 15, g = lane >> 4;
    const int wk = w % WK, we = (w / WK) % WE, wt = w / (WK * WE);
    const int t0 = blockIdx.x * TM + wt * 16;
    const XT* xrow = x + (size_t)min(t0 + n, T - 1) * d;           // A row of this lane (clamped, not stored)

    // k is cut into 32-row chunks; split s of the WK k-splits owns chunks [s*cper, (s+1)*cper).
    // In step c the work-group stages chunk s*cper + c of every split and each wave multiplies its
    // own split's tile.  Operands of the next kGPD steps are always in flight: all loads are
    // unconditional (addresses clamped, values zeroed when consumed), so no branch separates a load
    // from its use and the compiler can count outstanding loads exactly.
    const int chunks = (d + kGK - 1) / kGK;
    const int cper = (chunks + WK - 1) / WK;

    for (int e0 = 0; e0 < E; e0 += EN) {
        f32x4_t acc[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

        typedef float bword_t __attribute__((ext_vector_type(VEC)));
        bword_t breg[kGPD][NB];
        XRaw<XT> areg[kGPD];

        auto b_load = [&](bword_t (&dst)[NB], int c) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int p = (tid + i * 256) * VEC;
                const int s = p / (kGK * EN), kk = (p / EN) % kGK, ee = p % EN;
                const int k = min((s * cper + c) * kGK + kk, d - 1), e = min(e0 + ee, E - VEC);
                dst[i] = *reinterpret_cast<const bword_t*>(Wg + (size_t)k * E + e);
            }
        };
        auto b_store = [&](const bword_t (&src)[NB], int c) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int p = (tid + i * 256) * VEC;
                const int s = p / (kGK * EN), kk = (p / EN) % kGK, ee = p % EN;
                bword_t v = src[i];
                if (!FULL) {
                    const bool in = (s * cper + c) * kGK + kk < d && e0 + ee < E && c < cper;
#pragma unroll
                    for (int q = 0; q < VEC; ++q) v[q] = in ? v[q] : 0.f;
                }
                // columns rotated by 16 per 8 rows: the four lane groups of a B read hit distinct banks
                *reinterpret_cast<bword_t*>(&Bs[s][kk][(ee + 16 * (kk >> 3)) % EN]) = v;
            }
        };
        // one step: tile of chunk c to LDS, refill the register slot kGPD steps ahead, multiply
        auto step = [&](bword_t (&bslot)[NB], XRaw<XT>& aslot, int c) {
            lds_barrier();                            // the previous step has finished reading the tile
            b_store(bslot, c);
            float av[8];
            const int ka = (wk * cper + c) * kGK + 8 * g;
            aslot.widen(FULL ? 0 : (c < cper ? ka : d), d, av);
            lds_barrier();
            b_load(bslot, c + kGPD);
            aslot.load(xrow, (wk * cper + c + kGPD) * kGK + 8 * g, d);
            __builtin_amdgcn_sched_barrier(0);
            float bv[8][4];
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) bv[j][nt] = Bs[wk][8 * g + j][(we * 64 + nt * 16 + n + 16 * g) % EN];
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j], bv[j][nt], acc[nt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };

#pragma unroll
        for (int s = 0; s < kGPD; ++s) {
            b_load(breg[s], s);
            areg[s].load(xrow, (wk * cper + s) * kGK + 8 * g, d);
        }
        int c0 = 0;
        for (; c0 + kGPD <= cper; c0 += kGPD) {
#pragma unroll
            for (int s = 0; s < kGPD; ++s) step(breg[s], areg[s], c0 + s);
        }
        if (c0 < cper) step(breg[0], areg[0], c0);
        if (c0 + 1 < cper) step(breg[1], areg[1], c0 + 1);

        if constexpr (K > 0) {                       // one pass: E <= 64
            __shared__ int32_t e_sh[K * kLogitsTokens], h_sh[K * 64];
            __syncthreads();
            // partial sums of the rows that other waves finish: wave r finishes rows 4 g + r
            float own[4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    if (r != wk) red[((wk * 3 + (r < wk ? r : r - 1)) * 4 + nt) * 64 + lane] = acc[nt][r];
                    else own[nt] = acc[nt][r];
                }
            for (int i = tid; i < K * E; i += 256) h_sh[i] = 0;
            __syncthreads();
            const int tl = 4 * g + wk, t = t0 + tl;
            float v[4];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const int e = nt * 16 + n;
#pragma unroll
                for (int s = 0; s < 4; ++s) {        // in the order of the splits
                    const float p = s == wk ? own[nt] : red[((s * 3 + (wk < s ? wk : wk - 1)) * 4 + nt) * 64 + lane];
                    v[nt] = s == 0 ? p : v[nt] + p;
                }
                v[nt] += bg ? bg[min(e, E - 1)] : 0.f;
                if (t < T && e < E) logits[(size_t)t * E + e] = v[nt];
                v[nt] = e < E ? v[nt] : -INFINITY;
            }
            Best g1, g2;
            float w1, w2;
            token_gate_regs<K, 4>(v, E, n, g1, g2, w1, w2);
            if (n == 0) {
                e_sh[tl] = t < T ? g1.i : -1;
                if (K == 2) e_sh[kLogitsTokens + tl] = t < T ? g2.i : -1;
                if (t < T) {
                    expert_idx[(size_t)t * K] = g1.i;
                    gate_w[(size_t)t * K] = w1;
                    if (K == 2) {
                        expert_idx[(size_t)t * K + 1] = g2.i;
                        gate_w[(size_t)t * K + 1] = w2;
                    }
                }
            }
            __syncthreads();
            if (w == 0) {                            // one lane per token: rank among the tile's tokens with the same expert
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    const int e = lane < kLogitsTokens ? e_sh[j * kLogitsTokens + lane] : -1;
                    const int rank = wave_rank_by_expert(e, lane, E, h_sh + j * E);
                    if (e >= 0) slot_idx[(size_t)(t0 + lane) * K + j] = rank;
                }
            }
            __syncthreads();
            for (int i = tid; i < K * E; i += 256) hist[(size_t)blockIdx.x * K * E + i] = h_sh[i];
            // There is no second pass, but the compiler is not told: with `return` it keeps all addresses of a step in registers and moves
            // operands out of their way (moe_gate, 2500 tokens, d = 2048, 8 experts, top-2: 31.9 -> 30.1 us).
            continue;
        }
        if (WK > 1) {
            __syncthreads();
            float* mine = red + ((size_t)((wk - 1) * WT * WE + wt * WE + we) * 16) * 64;
            if (wk > 0) {
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mine[(nt * 4 + r) * 64 + lane] = acc[nt][r];
            }
            __syncthreads();
            if (wk == 0) {
                for (int s = 1; s < WK; ++s) {
                    const float* o = red + ((size_t)((s - 1) * WT * WE + wt * WE + we) * 16) * 64;
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[nt][r] += o[(nt * 4 + r) * 64 + lane];
                }
            }
        }
        if (wk == 0) {
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                const int e = e0 + we * 64 + nt * 16 + n;
                if (e >= E) continue;
                const float b = bg ? bg[e] : 0.f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int t = t0 + 4 * g + r;
                    if (t < T) logits[(size_t)t * E + e] = acc[nt][r] + b;
                }
            }
        }
        __syncthreads();      // the next expert pass restages the tile
    }
}

constexpr int kFewTokens = 4096;
template <typename XT>
static int launch_logits_t(const XT* x, const float* Wg, const float* bg, float* logits, int T, int d, int E,
                           hipStream_t s) {
#define MOE_LOGITS_CASE(WT, WE, WK)                                                                          \
    do {                                                                                                     \
        const dim3 grid((T + WT * 16 - 1) / (WT * 16));                                                      \
        const bool full = d % (kGK * WK) == 0 && E % (WE * 64) == 0;                                         \
        if (full)                                                                                            \
            hipLaunchKernelGGL((gate_logits_kernel<XT, WT, WE, WK, 4, true>), grid, dim3(256), 0, s, x, Wg, bg,     \
                               logits, T, d, E);                                                             \
        else if (E % 4 == 0)                                                                                 \
            hipLaunchKernelGGL((gate_logits_kernel<XT, WT, WE, WK, 4, false>), grid, dim3(256), 0, s, x, Wg, bg,    \
                               logits, T, d, E);                                                             \
        else                                                                                                 \
            hipLaunchKernelGGL((gate_logits_kernel<XT, WT, WE, WK, 1, false>), grid, dim3(256), 0, s, x, Wg, bg,    \
                               logits, T, d, E);                                                             \
    } while (0)
    const bool wide = E > 64;          // 128 experts per pass, else 64
    const bool few = T <= kFewTokens;  // few tokens: waves go to k-splits, not token tiles (1536 tokens, d = 512: 14.6 us without)
    if (wide) {
        if (few) MOE_LOGITS_CASE(1, 2, 2);
        else MOE_LOGITS_CASE(2, 2, 1);
    } else {
        if (few) MOE_LOGITS_CASE(1, 1, 4);
        else MOE_LOGITS_CASE(4, 1, 1);
    }
#undef MOE_LOGITS_CASE
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// Logits, top-k, tile-local ranks and histograms of 16 tokens each in one launch: few enough tokens that the waves go to k-splits,
// one pass of experts.  Fewer than 257 tokens have the whole routing in one work-group.  Of 150 shapes (260 to 4096 tokens, d 64 to 4096,
// 8, 31 and 64 experts) none is slower than with a launch for each, by 0.5 to 3.5 us; the finalising kernel's larger number of
// histograms does not show.
bool gate_logits_routes(int T, int E) { return T > kRouteTokens && T <= kFewTokens && E <= 64; }

template <typename XT>
static int launch_logits_route_t(const XT* x, const float* Wg, const float* bg, float* logits, int T, int d, int E, int k, int32_t* expert_idx,
                                 int32_t* slot_idx, float* gate_w, int32_t* hist, hipStream_t s) {
    const dim3 grid((T + kLogitsTokens - 1) / kLogitsTokens);
    const bool full = d % (kGK * 4) == 0 && E == 64;
#define MOE_LOGITS_CASE(vec, is_full, kk) \
    hipLaunchKernelGGL((gate_logits_kernel<XT, 1, 1, 4, vec, is_full, kk>), grid, dim3(256), 0, s, x, Wg, bg, logits, T, d, E, expert_idx, \
                       slot_idx, gate_w, hist)
    if (k == 1) {
        if (full) MOE_LOGITS_CASE(4, true, 1);
        else if (E % 4 == 0) MOE_LOGITS_CASE(4, false, 1);
        else MOE_LOGITS_CASE(1, false, 1);
    } else {
        if (full) MOE_LOGITS_CASE(4, true, 2);
        else if (E % 4 == 0) MOE_LOGITS_CASE(4, false, 2);
        else MOE_LOGITS_CASE(1, false, 2);
    }
#undef MOE_LOGITS_CASE
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}
int launch_gate_logits_route(const void* x, int dtype, const float* Wg, const float* bg, float* logits, int T, int d, int E, int k,
                             int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* scratch, int* tokens_per_hist, hipStream_t s) {
    if (!gate_logits_routes(T, E) || k < 1 || k > 2) return MOE_ERR_INVALID_ARG;
    *tokens_per_hist = kLogitsTokens;
    if (dtype == MOE_F32) return launch_logits_route_t(static_cast<const float*>(x), Wg, bg, logits, T, d, E, k, expert_idx, slot_idx, gate_w, scratch, s);
    return launch_logits_route_t(static_cast<const uint16_t*>(x), Wg, bg, logits, T, d, E, k, expert_idx, slot_idx, gate_w, scratch, s);
}

int launch_gate_logits(const void* x, int dtype, const float* Wg, const float* bg, float* logits, int T, int d,
                       int E, hipStream_t s) {
    if (dtype == MOE_F32) return launch_logits_t(static_cast<const float*>(x), Wg, bg, logits, T, d, E, s);
    return launch_logits_t(static_cast<const uint16_t*>(x), Wg, bg, logits, T, d, E, s);
}

// ------------------------------------------------------------------------------------------
// Routing, kernel 1 of 2, a block per TB tokens: top-k and gate weights, the rank of each token among the tile's
// tokens that chose the same expert (parked in slot_idx until kernel 2 adds the tile's base), the tile's histogram
// hist[tile][choice][E].  Latency-bound with few tokens, so tiles are small and many: blocks of 256 threads for 256 tokens
// (16 dependent rounds of top-k each) took 38.7 us for 777 tokens, 128 experts, top-2.  But every block of kernel 2 reads
// the histograms of all tiles, which grows with the square of T: from 32768 tokens on a tile has 256 tokens and 1024 threads.
// Both kernels, us, small tiles / tiles of 256: 64 experts, top-2, 32768 tokens 18.3 / 13.2, 131072 79 / 30; 128 experts,
// top-2, 8192 14.2 / 16.8, 16384 18.5 / 15.7, 262144 524 / 118; 512 experts 16384 61 / 71, 32768 78 / 77, 262144 755 / 387.
// ------------------------------------------------------------------------------------------
constexpr int kSmallRouteTiles = 32768;        // tokens below which tiles are small
template <int K, int NV, int TB>
__global__ __launch_bounds__(TB == kRouteTokens ? 1024 : 256) void route_tile_kernel(const float* __restrict__ logits, int T, int E,
                                                                                     int32_t* __restrict__ expert_idx,
                                                                                     int32_t* __restrict__ slot_idx,
                                                                                     float* __restrict__ gate_w,
                                                                                     int32_t* __restrict__ hist) {
    constexpr int NT = TB == kRouteTokens ? 1024 : 256, NW = (TB + kWave - 1) / kWave;    // waves that rank 64 tokens each
    static_assert(kRouteTokens % TB == 0, "whole tiles in a block of kernel 2");
    extern __shared__ int32_t smem[];
    int32_t* e_sh = smem;                          // [K][TB]
    int32_t* h_sh = smem + K * TB;                 // [NW][K][E]
    const int tid = threadIdx.x, t0 = blockIdx.x * TB, w = tid / kWave;
    for (int i = tid; i < NW * K * E; i += NT) h_sh[i] = 0;
    choose_experts<K, NV, NT, TB>(e_sh, logits, t0, min(TB, T - t0), T, E, expert_idx, gate_w);
    __syncthreads();
    int my_e[K], rank[K];
    if (tid < NW * kWave) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            my_e[j] = tid < TB ? e_sh[j * TB + tid] : -1;
            rank[j] = wave_rank_by_expert(my_e[j], tid % kWave, E, h_sh + (w * K + j) * E);
        }
    }
    __syncthreads();
    for (int i = tid; i < K * E; i += NT) {        // the tile's histogram, and the tokens of the waves before each
        int run = 0;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            const int c = h_sh[ww * K * E + i];
            h_sh[ww * K * E + i] = run;
            run += c;
        }
        hist[(size_t)blockIdx.x * K * E + i] = run;
    }
    __syncthreads();
    if (tid < TB) {
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (my_e[j] >= 0) slot_idx[(size_t)(t0 + tid) * K + j] = rank[j] + h_sh[(w * K + j) * E + my_e[j]];
    }
}

// ------------------------------------------------------------------------------------------
// Routing, kernel 2 of 2: every block sums the histograms of the blocks before it (its base)
// and of all blocks (totals), then turns block-local ranks into rows:
//   first choices:  row = base_1[e] + rank
//   second choices: row = total_1[e] + base_2[e] + rank      (all first choices rank first)
// row >= C -> dropped (-1).  Rows >= expert_rows[e] of slot_token are set to -1.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void expert_order_kernel(const int32_t* __restrict__ expert_rows, int E, int C,
                                                            int32_t* __restrict__ order) {
    extern __shared__ int32_t smem[];                 // rows, sorted and active experts: [E] each
    if (threadIdx.x < E) smem[threadIdx.x] = min(expert_rows[threadIdx.x], C);
    __syncthreads();
    write_expert_order(smem, E, order, smem + E, smem + 2 * E, threadIdx.x, blockDim.x);
}

int launch_expert_order(const int32_t* expert_rows, int E, int C, int32_t* order, hipStream_t s) {
    hipLaunchKernelGGL(expert_order_kernel, dim3(1), dim3(E <= 256 ? 256 : 1024), sizeof(int32_t) * 3 * E, s, expert_rows, E, C, order);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

constexpr int kFinThreads = 1024;   // at most; four times the tokens of a block: the sums over all tiles are most of its work

// row groups that share a column's sum: all threads, but few enough that adding up their results stays short
__host__ __device__ inline int finalize_row_groups(int ncol, int nthreads) {
    const int r = ncol >= nthreads ? 1 : nthreads / ncol;
    return r < 16 ? r : 16;
}

// hist holds one histogram [K][E] per block of TB tokens (TB divides 256, TB >= 16).  A work-group finalises 256
// tokens.  Every work-group sums the histograms of all blocks before its own: the reads grow with the square of the
// number of blocks (T = 16384, E = 64, top-2: 8 MB in all, served by L2), a stated limit of this kernel.
template <int K>
__device__ __forceinline__ void route_finalize_body(int32_t* smem, int T, int E, int C, int nblocks, int chunk, int TB,
                                                    const int32_t* __restrict__ expert_idx, int32_t* __restrict__ slot_idx,
                                                    int32_t* __restrict__ expert_rows, int32_t* __restrict__ slot_token,
                                                    int32_t* __restrict__ expert_order, const int32_t* __restrict__ hist) {
    const int ncol = K * E;                                // column = (choice j, expert e)
    const int q = kRouteTokens / TB;                       // fine blocks per work-group
    int32_t* base = smem;                                  // [q][K][E] rows before the fine block's tokens
    int32_t* rows_sh = base + q * ncol;                    // [E]
    int32_t* part = rows_sh + E;                           // [2][R][ncol]: before-me sums, all-blocks sums
    const int tid = threadIdx.x;
    const int b = blockIdx.x;

    // the tiles' histograms are summed with all threads: R row groups each take every R-th tile,
    // partial sums meet in LDS
    const int nt = blockDim.x, nfine = (T + TB - 1) / TB, R = finalize_row_groups(ncol, nt);
    for (int idx = tid; idx < R * ncol; idx += nt) {
        const int rg = (int)(((float)idx + 0.5f) * __builtin_amdgcn_rcpf((float)ncol)), col = idx - rg * ncol;   // idx < 2^12: exact
        int pre = 0, tot = 0;
        // every TB-token block's histogram once; those of 256-token blocks before this one also count as "before me"
        const int first_own = b * q;
        int fb = rg;
        // Fewer than 16 left: in powers of two, so that their loads are on their way together too (one after the other, moe_gate took
        // for 2500 fp32 tokens of 8 experts, d = 2048, top-2 30.3 us, now 28.4, the routing of 4096 given logits of 8 experts 9.2 and 7.5).
        auto add = [&](auto count) {                            // so many loads on their way at once
            constexpr int N = decltype(count)::value;
            int v[N];
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = hist[(size_t)(fb + i * R) * ncol + col];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                tot += v[i];
                pre += fb + i * R < first_own ? v[i] : 0;
            }
            fb += N * R;
        };
        const int left = nfine / R;                             // every row group has so many
#pragma unroll 16
        for (int n = left & ~15; n > 0; --n, fb += R) {
            const int v = hist[(size_t)fb * ncol + col];
            tot += v;
            pre += fb < first_own ? v : 0;
        }
        if (left & 8) add(std::integral_constant<int, 8>{});
        if (left & 4) add(std::integral_constant<int, 4>{});
        if (left & 2) add(std::integral_constant<int, 2>{});
        if (left & 1) add(std::integral_constant<int, 1>{});
        if (fb < nfine) add(std::integral_constant<int, 1>{});
        part[rg * ncol + col] = pre;
        part[(R + rg) * ncol + col] = tot;
    }
    // the histograms of this block's own tiles on the same memory round trip, turned into bases below
    for (int idx = tid; idx < q * ncol; idx += nt) {
        const long long at = (long long)b * q * ncol + idx;
        base[idx] = at < (long long)nfine * ncol ? hist[at] : 0;
    }
    __syncthreads();
    for (int col = tid; col < ncol; col += nt) {
        const int j = K == 2 && col >= E ? 1 : 0, e = col - j * E;
        int pre = 0, tot[K] = {};
#pragma unroll 8
        for (int rg = 0; rg < R; ++rg) {
            pre += part[rg * ncol + col];
#pragma unroll
            for (int i = 0; i < K; ++i) tot[i] += part[(R + rg) * ncol + i * E + e];
        }
        // first choices: rows before = first choices of earlier tokens; second choices rank behind ALL first ones
        int run = pre + (j == 1 ? tot[0] : 0);
        for (int f0 = 0; f0 < q; f0 += 4) {                     // four LDS reads at a time
            int v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = f0 + i < q ? base[(f0 + i) * ncol + col] : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (f0 + i < q) base[(f0 + i) * ncol + col] = run;
                run += v[i];
            }
        }
        if (j == 0) rows_sh[e] = min(tot[0] + (K == 2 ? tot[K - 1] : 0), C);
    }
    __syncthreads();

    const int t = b * kRouteTokens + tid;
    if (tid < kRouteTokens && t < T) {
        const int f = tid >> ceil_log2(TB);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int e = expert_idx[(size_t)t * K + j];
            const int loc = base[(f * K + j) * E + e] + slot_idx[(size_t)t * K + j];
            if (loc < C) {
                slot_idx[(size_t)t * K + j] = loc;
                slot_token[(size_t)e * C + loc] = t;
            } else {
                slot_idx[(size_t)t * K + j] = -1;
            }
        }
    }

    const long long lo = (long long)b * chunk;                   // chunk: a block's share of the E C entries
    const long long hi = min(lo + chunk, (long long)E * C);
    for (uint32_t i = (uint32_t)lo + tid; i < hi; i += nt)        // E * C < 2^31
        if ((int)(i % (uint32_t)C) >= rows_sh[i / (uint32_t)C]) slot_token[i] = -1;
    // The rows per expert and the launch order are the work of one block: with an order to write, of an extra block
    // behind the last one (no tokens, no slots: everything above ran empty for it), so that the ranking does not
    // lengthen a block that also has tokens to place.
    if (b == (expert_order ? nblocks : 0)) {
        for (int e = tid; e < E; e += nt) expert_rows[e] = rows_sh[e];
        if (expert_order) write_expert_order(rows_sh, E, expert_order, part, part + E, tid, nt);   // part: free by now
    }
}

template <int K>
__global__ __launch_bounds__(kFinThreads) void route_finalize_kernel(int T, int E, int C, int nblocks, int chunk, int TB,
                                                                      const int32_t* __restrict__ expert_idx,
                                                                      int32_t* __restrict__ slot_idx,
                                                                      int32_t* __restrict__ expert_rows,
                                                                      int32_t* __restrict__ slot_token,
                                                                      int32_t* __restrict__ expert_order,
                                                                      const int32_t* __restrict__ hist) {
    extern __shared__ int32_t smem[];
    route_finalize_body<K>(smem, T, E, C, nblocks, chunk, TB, expert_idx, slot_idx, expert_rows, slot_token, expert_order, hist);
}

// At most 256 tokens (decode): one block, whose local ranks are already global ones -- the whole routing in one
// launch with a single memory round trip (the logits): totals and ranks stay in LDS and registers.
template <int K, int NV>
__global__ __launch_bounds__(kSingleThreads) void route_single_kernel(const float* __restrict__ logits, int T, int E, int C,
                                                                    int32_t* __restrict__ expert_idx,
                                                                    int32_t* __restrict__ slot_idx,
                                                                    float* __restrict__ gate_w,
                                                                    int32_t* __restrict__ expert_rows,
                                                                    int32_t* __restrict__ slot_token,
                                                                    int32_t* __restrict__ expert_order) {
    extern __shared__ int32_t smem[];
    route_single_body<K, NV>(smem, logits, T, E, C, expert_idx, slot_idx, gate_w, expert_rows, slot_token, expert_order);
}

size_t route_finalize_lds_bytes(int E, int k, int TB, int nthreads) {
    const int ncol = k * E;
    const int R = finalize_row_groups(ncol, nthreads);
    const size_t ints = (size_t)(kRouteTokens / TB) * ncol + E + 2 * (size_t)R * ncol;   // the last part: 2 E for the launch order
    return ints * sizeof(int32_t);
}

int launch_route_finalize(int T, int E, int k, int C, int TB, const int32_t* expert_idx, int32_t* slot_idx,
                          int32_t* expert_rows, int32_t* slot_token, int32_t* expert_order, const int32_t* hist,
                          hipStream_t s) {
    const int nb = (T + kRouteTokens - 1) / kRouteTokens;
    // Many tokens and few columns: little to add up per block, and small blocks are more of them on the chip at once (top-1, both
    // kernels, 1024 / 256 threads: 8 experts, 524288 tokens 56 / 34 us; 64 experts, 98304 20.4 / 16.2, 524288 107 / 90; top-2 of
    // 128 experts, 65536 21.7 / 24.6).
    const int nt = T >= kSmallRouteTiles && k * E <= 64 ? 256 : kFinThreads;
    const size_t sm = route_finalize_lds_bytes(E, k, TB, nt);
    const int chunk = (int)(((long long)E * C + nb - 1) / nb);
    const int grid = nb + (expert_order ? 1 : 0);               // + the block that ranks the experts
    if (k == 1)
        hipLaunchKernelGGL((route_finalize_kernel<1>), dim3(grid), dim3(nt), sm, s, T, E, C, nb, chunk, TB, expert_idx,
                           slot_idx, expert_rows, slot_token, expert_order, hist);
    else
        hipLaunchKernelGGL((route_finalize_kernel<2>), dim3(grid), dim3(nt), sm, s, T, E, C, nb, chunk, TB, expert_idx,
                           slot_idx, expert_rows, slot_token, expert_order, hist);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// histograms for blocks of 32 tokens at the finest, of 16 where gate_logits_kernel writes them; no less than for fewer tokens
size_t route_scratch_ints(int T, int E, int k, bool by_logits) {
    size_t fine = ((size_t)T + 31) / 32;
    const int few = T < kFewTokens ? T : kFewTokens;
    if (by_logits && gate_logits_routes(few, E)) {
        const size_t tiles = (few + kLogitsTokens - 1) / kLogitsTokens;
        fine = fine < tiles ? tiles : fine;
    }
    return fine * (size_t)k * (size_t)E;
}

int launch_route(const float* logits, int T, int E, int k, int C, int32_t* expert_idx, int32_t* slot_idx,
                 float* gate_w, int32_t* expert_rows, int32_t* slot_token, int32_t* expert_order, int32_t* scratch,
                 hipStream_t s) {
    if (T <= kRouteTokens) {
        const size_t sm = route_single_lds_ints(E, k) * sizeof(int32_t);
#define MOE_ROUTE_SINGLE(K, NV)                                                                                        \
    hipLaunchKernelGGL((route_single_kernel<K, NV>), dim3(1), dim3(kSingleThreads), sm, s, logits, T, E, C, expert_idx, \
                       slot_idx, gate_w, expert_rows, slot_token, expert_order)
        if (k == 1) {
            if (E <= 16) MOE_ROUTE_SINGLE(1, 1);
            else if (E <= 32) MOE_ROUTE_SINGLE(1, 2);
            else if (E <= 64) MOE_ROUTE_SINGLE(1, 4);
            else if (E <= 128) MOE_ROUTE_SINGLE(1, 8);
            else MOE_ROUTE_SINGLE(1, 0);
        } else {
            if (E <= 16) MOE_ROUTE_SINGLE(2, 1);
            else if (E <= 32) MOE_ROUTE_SINGLE(2, 2);
            else if (E <= 64) MOE_ROUTE_SINGLE(2, 4);
            else if (E <= 128) MOE_ROUTE_SINGLE(2, 8);
            else MOE_ROUTE_SINGLE(2, 0);
        }
#undef MOE_ROUTE_SINGLE
        return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
    }
    const int TB = T >= kSmallRouteTiles ? kRouteTokens : E <= 128 ? 32 : 64;   // E > 128: kernel 2 keeps k E 256 / TB sums in LDS
    const size_t sm = sizeof(int32_t) * ((size_t)k * TB + (size_t)((TB + kWave - 1) / kWave) * k * E);
    const unsigned tiles = (unsigned)((T + TB - 1) / TB);
#define MOE_ROUTE_TILE(K, NV)                                                                                             \
    do {                                                                                                                  \
        if (TB == kRouteTokens)                                                                                           \
            hipLaunchKernelGGL((route_tile_kernel<K, NV, kRouteTokens>), dim3(tiles), dim3(1024), sm, s, logits, T, E,    \
                               expert_idx, slot_idx, gate_w, scratch);                                                    \
        else                                                                                                              \
            hipLaunchKernelGGL((route_tile_kernel<K, NV, (NV > 0 ? 32 : 64)>), dim3(tiles), dim3(256), sm, s, logits, T,  \
                               E, expert_idx, slot_idx, gate_w, scratch);                                                 \
    } while (0)
    if (k == 1) {
        if (E <= 16) MOE_ROUTE_TILE(1, 1);
        else if (E <= 32) MOE_ROUTE_TILE(1, 2);
        else if (E <= 64) MOE_ROUTE_TILE(1, 4);
        else if (E <= 128) MOE_ROUTE_TILE(1, 8);
        else MOE_ROUTE_TILE(1, 0);
    } else {
        if (E <= 16) MOE_ROUTE_TILE(2, 1);
        else if (E <= 32) MOE_ROUTE_TILE(2, 2);
        else if (E <= 64) MOE_ROUTE_TILE(2, 4);
        else if (E <= 128) MOE_ROUTE_TILE(2, 8);
        else MOE_ROUTE_TILE(2, 0);
    }
#undef MOE_ROUTE_TILE
    if (hipGetLastError() != hipSuccess) return MOE_ERR_HIP;
    return launch_route_finalize(T, E, k, C, TB, expert_idx, slot_idx, expert_rows, slot_token, expert_order,
                                 scratch, s);
}

}  // namespace moe
