// Internal declarations shared by the library's translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "moe.h"
#include "once_per_device.h"

namespace moe {

constexpr int kWave = 64;            // CDNA wavefront width
constexpr int kRouteTokens = 256;    // tokens per block in the routing kernels

// Leave for a kernel to be launched with so much dynamic LDS, which takes a call per device beyond 64 KB; asked: one per kernel.
inline int ask_lds(const void* kernel, int bytes, OncePerDevice& asked) {
    if (bytes <= 64 * 1024) return MOE_OK;
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return MOE_ERR_HIP;
    auto ask = [=] { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess; };
    return asked(device, ask) ? MOE_OK : MOE_ERR_HIP;
}

// Work-group barrier that orders LDS traffic only.  __syncthreads() also drains every outstanding
// global load (on gfx9 loads and stores share one counter), which would empty the register prefetch
// queues the streaming kernels depend on at each barrier.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- bf16 <-> f32 on raw 16-bit patterns -------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t v) {
    return __uint_as_float(static_cast<uint32_t>(v) << 16);
}
// round to nearest even; NaN stays NaN
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}
// two fp32 -> packed bf16, round to nearest even, on the hardware converter (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const bf16x2_t v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
    return __builtin_bit_cast(uint32_t, v);
}
// M pairs of fp32 values as three times M pairs of bf16: a value is piece 0 + piece 1 + piece 2 (3 x 8 significant bits, each piece the
// nearest bf16 of what is left), exactly as long as the pieces are not below bf16's 2^-133.  x holds what is left before the last piece.
template <int M> __device__ __forceinline__ void split_bf16x3(float (&x)[M][2], uint32_t (&piece)[3][M]) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {                            // piece by piece, so that no instruction waits for the one before it
#pragma unroll
        for (int i = 0; i < M; ++i) {
            piece[q][i] = pack_bf16x2(x[i][0], x[i][1]);
            asm("" : "+v"(piece[q][i]));                     // one conversion for both values, not one more for the first alone
        }
        if (q == 2) break;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            x[i][0] -= __uint_as_float(piece[q][i] << 16);
            x[i][1] -= __uint_as_float(piece[q][i] & 0xffff0000u);
        }
    }
}

// gelu_tanh(z) = 0.5 z (1 + tanh(u)), u = sqrt(2/pi) (z + 0.044715 z^3).  Since tanh(u) = 2 sigmoid(2u) - 1 this is
// z sigmoid(2u) = z / (1 + exp(-2u)): one exp2 and one rcp on the hardware units, five multiply-adds.
constexpr float kGelu1 = -2.3022082f, kGelu3 = -0.10294324f;   // -2u log2(e) = z (kGelu1 + kGelu3 z^2)
__device__ __forceinline__ float gelu_tanh(float z) {
    const float z2 = z * z;
    const float e = __builtin_amdgcn_exp2f(z * fmaf(z2, kGelu3, kGelu1));
    return z * __builtin_amdgcn_rcpf(1.0f + e);
}

// zero(t, lane) by a whole wave for every token t < T whose first choice has no slot; 16 tokens per wave at a time, dealt to
// the work-groups first and to their waves then.
template <typename F>
__device__ __forceinline__ void for_dropped_tokens(const int32_t* slot_idx, int top_k, int T, int tid, int nthreads, F zero) {
    const int lane = tid % kWave;
    const long long blocks = (long long)gridDim.x * gridDim.y, block = (long long)blockIdx.y * gridDim.x + blockIdx.x;
    const int pieces = (int)(((long long)T + 15) / 16);
    for (long long c = block + blocks * __builtin_amdgcn_readfirstlane(tid / kWave); c < pieces; c += blocks * (nthreads / kWave)) {
        const int t0 = (int)c * 16;
        const bool dropped = lane < 16 && t0 + lane < T && slot_idx[(size_t)(t0 + lane) * top_k] < 0;
        for (unsigned long long m = __ballot(dropped); m; m &= m - 1) zero(t0 + __ffsll((long long)m) - 1, lane);
    }
}

// ---- sums of a product whose K was split, added up by the kernel that reads them next -------
constexpr int kLinearMaxSplit = 8;   // parts at most
struct PartSums {
    const float* partial;      // [ksplit, T, d], or nullptr: none
    int32_t ksplit;
    const uint16_t* bias;      // [d] in bf16, or nullptr
};

// v = elements 8 i .. 8 i + 7 of the row at `row` (T d elements per part): the parts in order, then the bias; all loads first
__device__ __forceinline__ void add_parts8(const PartSums& s, size_t part, size_t row, int i, float (&v)[8]) {
    float4 p[kLinearMaxSplit][2];
#pragma unroll
    for (int n = 0; n < kLinearMaxSplit; ++n)
#pragma unroll
        for (int q = 0; q < 2; ++q)
            p[n][q] = n < s.ksplit ? reinterpret_cast<const float4*>(s.partial + n * part + row)[2 * i + q] : make_float4(0.f, 0.f, 0.f, 0.f);
    const uint4 bias = s.bias ? reinterpret_cast<const uint4*>(s.bias)[i] : make_uint4(0, 0, 0, 0);
    // from the first part on: a sum that starts at 0 waits for it before the others' loads
    *reinterpret_cast<float4*>(v) = p[0][0];
    *reinterpret_cast<float4*>(v + 4) = p[0][1];
#pragma unroll
    for (int n = 1; n < kLinearMaxSplit; ++n) {
        if (n >= s.ksplit) break;
        v[0] += p[n][0].x; v[1] += p[n][0].y; v[2] += p[n][0].z; v[3] += p[n][0].w;
        v[4] += p[n][1].x; v[5] += p[n][1].y; v[6] += p[n][1].z; v[7] += p[n][1].w;
    }
    v[0] += __uint_as_float(bias.x << 16); v[1] += __uint_as_float(bias.x & 0xffff0000u);
    v[2] += __uint_as_float(bias.y << 16); v[3] += __uint_as_float(bias.y & 0xffff0000u);
    v[4] += __uint_as_float(bias.z << 16); v[5] += __uint_as_float(bias.z & 0xffff0000u);
    v[6] += __uint_as_float(bias.w << 16); v[7] += __uint_as_float(bias.w & 0xffff0000u);
}

// ---- launchers (each returns MOE_OK or MOE_ERR_HIP) ---------------------------------------

// logits[t,e] = bg[e] + sum_i x[t,i] Wg[i,e]
int launch_gate_logits(const void* x, int dtype, const float* Wg, const float* bg, float* logits,
                       int T, int d, int E, hipStream_t s);

// the same and, for few tokens and experts, the top-k, tile-local ranks (parked in slot_idx) and histograms in the same launch;
// launch_route_finalize(..., *tokens_per_hist, ..., scratch) completes the routing
bool gate_logits_routes(int T, int E);
int launch_gate_logits_route(const void* x, int dtype, const float* Wg, const float* bg, float* logits, int T, int d, int E, int k,
                             int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* scratch, int* tokens_per_hist, hipStream_t s);

// the same for bf16 tokens on the bf16 matrix cores (fp32 weights split into three bf16 pieces, exact); Wg_packed: the pieces as
// launch_pack_gate wrote them, or nullptr: Wg
bool gate_bf16_supported(int d, int E);
size_t gate_bf16_ws_bytes(int d, int E);
int launch_gate_logits_bf16(const void* x, const float* Wg, const void* Wg_packed, const float* bg, float* logits, int T,
                            int d, int E, hipStream_t s);
// the split weights written once into a caller-owned buffer of gate_bf16_ws_bytes(d, E) bytes (Wg_packed above)
int launch_pack_gate(const float* Wg, void* packed, int d, int E, hipStream_t s);

// logits, top-k, gate weights, tile-local ranks (parked in slot_idx) and per-tile histograms for bf16 tokens;
// launch_route_finalize(..., *tokens_per_hist, ..., *hist_out) completes the routing.
// frag_ws: gate_bf16_ws_bytes(d, E) bytes of scratch for the split weights, rewritten by every call without Wg_packed;
// scratch as for launch_route; logits is always written
bool gate_bf16_fused_supported(int T, int d, int E);
int launch_gate_bf16_fused(const void* x, const float* Wg, const void* Wg_packed, const float* bg, float* logits, int T,
                           int d, int E, int k, int32_t* expert_idx, int32_t* slot_idx, float* gate_w, void* frag_ws,
                           int32_t* scratch, int* tokens_per_hist, const int32_t** hist_out, hipStream_t s);

// the whole gate of at most 256 bf16 tokens in one launch (logits by many work-groups, routing by the last one);
// flags: kGateFlags words of scratch that may hold anything; tag: next_call_tag()
constexpr int kGateFlags = 64;
bool gate_decode_supported(int T, int d, int E);
int launch_gate_decode(const void* x, const float* Wg, const void* Wg_packed, const float* bg, float* logits, int T, int d,
                       int E, int k, int C, int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* expert_rows,
                       int32_t* slot_token, int32_t* expert_order, uint64_t* flags, uint64_t tag, hipStream_t s);

// number of int32 the routing kernels need as scratch
size_t route_scratch_ints(int T, int E, int k, bool by_logits /* tokens or shapes that the bf16 gate kernels do not take */);

// softmax + top-k + capacity slots from fp32 logits
int launch_route(const float* logits, int T, int E, int k, int C,
                 int32_t* expert_idx, int32_t* slot_idx, float* gate_w,
                 int32_t* expert_rows, int32_t* slot_token, int32_t* expert_order /* [2E + 2] or nullptr */,
                 int32_t* scratch, hipStream_t s);

// second routing kernel alone: hist = one histogram [k][E] per block of TB tokens (TB divides 256) with the
// block-local ranks parked in slot_idx
int launch_route_finalize(int T, int E, int k, int C, int TB, const int32_t* expert_idx, int32_t* slot_idx,
                          int32_t* expert_rows, int32_t* slot_token, int32_t* expert_order, const int32_t* hist,
                          hipStream_t s);

// the two launch orders of the experts (2E + 2 ints: see write_expert_order) from the row counts alone
int launch_expert_order(const int32_t* expert_rows, int E, int C, int32_t* order, hipStream_t s);

int launch_dispatch(const void* x, int dtype, const int32_t* slot_token, const int32_t* expert_rows,
                    void* xe, int E, int C, int d, hipStream_t s);

int launch_combine(const void* ye, int dtype, const int32_t* expert_idx, const int32_t* slot_idx,
                   const float* gate_w, const void* addend, void* out,
                   int T, int k, int C, int d, hipStream_t s,
                   const PartSums& dense = PartSums{});

// What a grouped GEMM does with a finished row.
enum WsEpilogue {
    EPI_STORE = 0,    // out[g*o_group_stride + r, :] = acc + bias
    EPI_GELU = 1,     // out[g*o_group_stride + r, :] = gelu_tanh(acc + bias)
    EPI_SCATTER = 2,  // out[token(g,r), :] = gate_w[token, 0] * (acc + bias)        (top-1 combine)
    EPI_COMBINE = 3,  // out[r, :] = acc + bias + sum_j keep_j g_j ye[e_j, slot_j, :]   (dense branch + combine)
    EPI_PARTIAL = 4   // partial[ks, g*o_group_stride + r, :] = acc   (split-K, fp32, no bias)
};
// fp32 grouped GEMM on the fp32 matrix cores (gemm_f32.hip); K and N multiples of 4, no EPI_PARTIAL.
struct GemmArgs {
    const void* A;            // activations, row-major, leading dimension K
    const void* B;            // [G, K, N] weights
    const void* bias;         // [G, N] or nullptr
    void* out;                // row-major, leading dimension N
    const int32_t* rows;      // [G] device row counts, or nullptr -> fixed_rows for every group
    const int32_t* row_map;   // [G, max_rows] A-row index per (g, r), or nullptr
    int32_t fixed_rows;
    int32_t max_rows;         // upper bound of rows(g): sizes the grid
    int32_t expect_rows;      // rows of a group if the tokens fall evenly on them; 0: max_rows
    int32_t G, K, N;
    int64_t a_group_stride;   // in rows; A-row of (g, r) = g*a_group_stride + r when row_map == nullptr
    int64_t o_group_stride;   // in rows; out-row of (g, r) = g*o_group_stride + r
    // EPI_SCATTER
    const int32_t* scatter_map;    // [G, max_rows] token per expert row
    int32_t T;                     // tokens; those with slot_idx < 0 get zero rows (top_k == 1)
    // EPI_SCATTER / EPI_COMBINE
    const float* gate_w;           // [T, top_k]
    const int32_t* slot_idx;       // [T, top_k]
    int32_t top_k;
    // EPI_COMBINE
    const void* ye;                // [E, C, N]
    const int32_t* expert_idx;     // [T, top_k]
    int32_t C;
};
int launch_gemm_f32(const GemmArgs& a, int epi, hipStream_t s);
// which kernel that is (gemm_f32.hip), for the dispatch report
enum F32Kernel {
    F32_ROWS16 = 1, F32_ROWS32 = 2,              // f32_rows_kernel, tiles of 16 and 32 rows
    F32_ROWS_SPLIT8 = 3, F32_ROWS_SPLIT4 = 4,    // f32_rows_split_kernel, eight and four waves
    F32_TILE_NARROW = 5, F32_TILE = 6,           // f32_tile_kernel, 128 x 64 and 64 x 128
    F32_SPLIT1 = 7, F32_SPLIT2 = 8,              // f32_split_kernel, one and two sets of waves
    F32_FFN = 9                                  // f32_ffn_kernel: both products
};
F32Kernel f32_kernel(const GemmArgs& a);
// both products of an FFN in one launch: a is the first, b the second on its output (a.out and b.A are not used); epi: the second's
bool ffn_f32_fused(const GemmArgs& a);
int launch_ffn_f32(const GemmArgs& a, const GemmArgs& b, int epi, hipStream_t s);

// bf16 MFMA weight-streaming grouped GEMM (ffn_mfma.hip).
struct WsGemmArgs {
    const uint16_t* A;         // activations, leading dimension K
    const uint16_t* B;         // [G, K, N], or the same weights in fragment order (packed != 0)
    int32_t stream;            // four-wave tile kernel: weights that only one row tile reads are not worth caching
    int32_t packed;            // B is [G, ceil(K/32), ceil(N/128), 8, 64, 8] as written by launch_pack_weights
    const uint16_t* bias;      // [G, N] or nullptr
    const int32_t* rows;       // [G] device row counts or nullptr -> fixed_rows
    const int32_t* order;      // [G + 1] groups in launch order (busiest first), then 2 * (groups that have rows) + the tile-dealing flag; or nullptr -> identity
    const int32_t* row_map;    // [G, map_stride]: A-row of (g, r), or nullptr -> g*a_group_stride + r
    int32_t fixed_rows, max_rows, map_stride;
    int32_t expect_rows;       // tiled kernel: rows of a group if the tokens fall evenly on them; 0: max_rows
    int32_t G, K, N;
    int32_t slots;             // entries of `order` that may have rows (the others certainly have none); 0: all
    long long a_group_stride;
    uint16_t* out;             // leading dimension N
    long long o_group_stride;
    int32_t ksplit;            // >= 1; > 1 only with EPI_PARTIAL
    int32_t split_tiles;       // with `order`: so many waves' tiles are enough, ksplit is the most (live_split); 0: always ksplit
    int32_t spread;            // tiled kernel, tile dealing: 0 = as order[G] says, 1 = always spread, 2 = never
    float* partial;            // [ksplit, partial_rows, N]
    long long partial_rows;
    // EPI_SCATTER
    const int32_t* scatter_map;    // [G, scatter_stride] token per expert row
    int32_t scatter_stride;
    const int32_t* zero_slot_idx;  // [T*top_k]: rows t with zero_slot_idx[t*top_k] < 0 are zero-filled (top_k == 1)
    int32_t T;
    // EPI_SCATTER / EPI_COMBINE
    const uint16_t* add;           // streaming and few-weights kernels: [T, N] rows that the results are added to, or nullptr
    const float* gate_w;           // [T, top_k]
    int32_t top_k;
    const uint16_t* ye;            // [E, C, N]
    const int32_t* expert_idx;     // [T, top_k]
    const int32_t* slot_idx;       // [T, top_k]
    int32_t C;
};
bool wsgemm_supported(int K, int N);
void wsgemm_pick_tile(int max_rows, int G, int N, int* MT, int* NW);
int launch_wsgemm(const WsGemmArgs& a, int epi, int MT, int NW, int NBUF, hipStream_t s);
int wsgemm_chunk_k(int MT);   // k-extent of one LDS chunk = granularity of split-K

// Products that read few weights (ffn_rows.hip): 16 NF columns per work-group, K split over its waves; ksplit must be 1.
// b: a second product of the same K, N and packing in the same launch (not with EPI_SCATTER), or nullptr.
int launch_rows(const WsGemmArgs& a, const WsGemmArgs* b, int epi, int NF, hipStream_t s);
// NF for a product, or 0 where another kernel does better.  touched: experts that can have rows; kept: rows of all of them
int rows_pick_gemm1(long long touched, int max_rows, long long kept, int K, int N, bool packed, bool with_dense);
int rows_pick_gemm2(int E, long long touched, int max_rows, long long kept, int K, int N, bool packed, bool few_waves);
int rows_pick_dense(int T, int N, bool packed);

// Tiled variant for groups with many rows (ffn_tile.hip); same arguments, ksplit must be 1.
int launch_tgemm(const WsGemmArgs& a, int epi, hipStream_t s);
// two grouped products in one launch (same K, N, packing, epilogue): more tiles, one shape for both
bool tgemm_pair_fusable(const WsGemmArgs& a, const WsGemmArgs& b);
int launch_tgemm_pair(const WsGemmArgs& a, const WsGemmArgs& b, int epi, hipStream_t s);
bool tgemm_supported(int K, int N);
// the kernel that these products get: 1000 rows + columns of its tiles; + 1: two work-groups per CU; + 2: the four-wave kernel,
// weights through the caches, + 3: with the non-temporal hint, + 4: as each group needs it
int tgemm_code(const WsGemmArgs& a, const WsGemmArgs* b, int epi);

// 256-column tiles of 256 or 128 rows on packed weights (ffn_wide.hip); b: a second product in the launch, or nullptr
int launch_wide(const WsGemmArgs& a, const WsGemmArgs* b, int tile_rows, int epi, hipStream_t s);
int wide_policy(const WsGemmArgs& a, const WsGemmArgs* b, int tile_rows, int epi);   // how it reads the weights (WidePolicy)

// Weights in the fragment order of v_mfma_f32_16x16x32_bf16's second operand (pack.hip).  Element (k, n) of group g
// goes to  ((((g*KB + k/32)*NG + n/128)*8 + n%8)*64 + (k%32/8)*16 + (n%128)/8)*8 + k%8,  KB = ceil(K/32),
// NG = ceil(N/128); positions past K or N hold zeros.  A lane's 16 bytes are then 8 consecutive k of one column,
// a wave's 1 KB is one fragment, and fragment j of a 128-column group holds columns 8c + j (c = lane % 16): a lane's
// 8 accumulators of a row are 8 consecutive columns.
inline size_t packed_weight_elems(int G, int K, int N) {
    return (size_t)G * ((K + 31) / 32) * ((N + 127) / 128) * 4096;
}
int launch_pack_weights(const uint16_t* W, uint16_t* packed, int G, int K, int N, hipStream_t s);

// Sums split-K partials in split order, adds the bias and finishes like EPI_STORE (scatter_map ==
// nullptr) or EPI_SCATTER (scatter_map given; also zero-fills rows of dropped tokens).
struct SplitKReduceArgs {
    const float* partial;      // [ksplit, G*group_stride, N]
    int32_t ksplit, G, N;
    const int32_t* order;      // with split_tiles: as the product that wrote the partials had them
    int32_t split_tiles;
    long long group_stride;
    const int32_t* rows;       // [G], or nullptr: max_rows for every group
    int32_t max_rows;
    const uint16_t* bias;      // [G, N] or nullptr
    uint16_t* out;
    const int32_t* scatter_map;
    const uint16_t* add;       // with scatter_map: [T, N] rows that the results are added to, or nullptr
    const float* gate_w;
    int32_t top_k;
    const int32_t* zero_slot_idx;
    int32_t T;
};
int launch_splitk_reduce(const SplitKReduceArgs& a, hipStream_t s);

// ---- the non-expert half of a decoder block, one decode step (block.hip) --------------------------------------
struct AddedRows {             // what a LayerNorm adds to its rows first: nothing, [T, d] rows, or a product's sums
    const uint16_t* rows;
    PartSums sums;             // only where add_layernorm_sums(d)
};
bool add_layernorm_sums(int d);
int launch_add_layernorm(const uint16_t* x, const AddedRows& r, const float* gamma, const float* beta,
                         uint16_t* sum_out /* x + r, or nullptr */, uint16_t* y, int T, int d, float eps, hipStream_t s);
int launch_add_rows(const uint16_t* a, const uint16_t* b, uint16_t* out, long long n, hipStream_t s);
bool attn_supported(int d, int H);
size_t attn_partial_floats(int T, int H, int dh, int Lmax);
int launch_attn_decode(const uint16_t* qkv, uint16_t* cache_k, uint16_t* cache_v, const int32_t* pos, float* partial,
                       uint16_t* attn, int T, int H, int dh, int Lmax, hipStream_t s);

}  // namespace moe
