// Pieces shared by the two bf16 MFMA grouped-GEMM kernels (weight-streaming and tiled): operand
// types, the register transpose of K-major weights, the XCD-aware tile numbering and the epilogues.
#pragma once

#include "moe_internal.h"

namespace moe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kXcd = 8;             // L2 domains; consecutive work-group ids rotate over them

__device__ __forceinline__ uint32_t dw(const uint4& v, int q) {
    return q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w;
}

// MFMA B fragments from K-major weights.  src[j] holds 8 consecutive columns of k-row j (j = 0..7):
// an 8x8 block of 16-bit values, k down, n across.  The MFMA wants, per output column, 8 consecutive
// k in one register quad: an 8x8 transpose, done with v_perm_b32.  Pair qq of the block's columns
// (2qq, 2qq+1) comes out as two fragments.
__device__ __forceinline__ void b_frag_pair(const uint4 (&src)[8], int qq, bf16x8_t& lo_col, bf16x8_t& hi_col) {
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t r0 = dw(src[2 * p], qq), r1 = dw(src[2 * p + 1], qq);
        lo[p] = __builtin_amdgcn_perm(r1, r0, 0x05040100u);   // column 2qq   : k = 2p, 2p+1
        hi[p] = __builtin_amdgcn_perm(r1, r0, 0x07060302u);   // column 2qq+1
    }
    lo_col = __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
    hi_col = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
}

// Consecutive work-group ids rotate over the 8 XCDs (each with its own L2).  With at least 8
// groups, all tiles of one expert are placed on one XCD: its activation rows (read by every
// column tile) and its weights (read by every row tile) are then fetched into that L2 once.
// Experts are taken from `order` (busiest first), dealt round-robin to the XCDs, so that each
// XCD streams the same number of active experts.  With fewer groups (the dense branch) column
// tiles are spread over the XCDs instead.  inner_n = row tiles x k-splits per (group, column tile).
struct TileId {
    int g, nt, inner;
    bool live;
};
__host__ __device__ __forceinline__ TileId tile_of_block(const WsGemmArgs& a, int n_tiles, int inner_n, int block) {
    TileId t;
    const int xcd = block % kXcd;
    const int q = block / kXcd;
    if (a.G >= kXcd) {
        const int per_group = n_tiles * inner_n;
        const int slot = (q / per_group) * kXcd + xcd;
        t.nt = (q % per_group) / inner_n;
        t.inner = q % inner_n;
        t.live = slot < a.G;
        t.g = t.live ? (a.order ? a.order[slot] : slot) : 0;
    } else if (a.ksplit == 1 && inner_n >= kXcd) {
        // few groups with many row tiles (the dense branch): every XCD takes a contiguous range of
        // row tiles and walks it column tile by column tile, so the work-groups running together on
        // an XCD share a few activation row tiles (kept in its L2) while the weights stream through
        const int per_xcd = (inner_n + kXcd - 1) / kXcd;
        const int per_group = per_xcd * n_tiles;
        t.g = q / per_group;
        t.nt = q % n_tiles;
        t.inner = xcd * per_xcd + (q % per_group) / n_tiles;
        t.live = t.g < a.G && t.inner < inner_n;
    } else {
        const int u = (q / inner_n) * kXcd + xcd;
        t.g = u / n_tiles;
        t.nt = u % n_tiles;
        t.inner = q % inner_n;
        t.live = u < a.G * n_tiles;
    }
    return t;
}
// Second mapping, for the tiled kernel with many groups of very different sizes (config 5: a few experts at capacity,
// many with a handful of rows): every XCD takes 1/8 of the column tiles of EVERY group and walks the groups in launch
// order, row tiles innermost.  All XCDs then carry the same work whatever the row counts are; a weight column tile
// still enters exactly one L2 (its row tiles run back to back there); only the groups' activation rows are read by
// all eight.  Because the launch order alternates busy and light groups, the CUs of an XCD run matrix-bound and
// weight-streaming tiles at the same time, instead of one phase after the other.
// Which mapping applies is decided on the device, by the flag (bit 0) behind the launch order (only the device knows the row
// counts); the host sizes the grid for either.
__host__ __device__ __forceinline__ bool tile_spread_possible(const WsGemmArgs& a, int n_tiles) {
    return a.order != nullptr && a.spread != 2 && a.ksplit == 1 && a.G >= kXcd && n_tiles % kXcd == 0;
}
__device__ __forceinline__ bool tile_spread(const WsGemmArgs& a, int n_tiles) {
    return tile_spread_possible(a, n_tiles) && (a.spread == 1 || (a.order[a.G] & 1));
}
__device__ __forceinline__ TileId tile_of_block_spread(const WsGemmArgs& a, int n_tiles, int inner_n, int block) {
    TileId t;
    const int xcd = block % kXcd, q = block / kXcd;
    const int per_x = n_tiles / kXcd, per_group = per_x * inner_n;
    const int slot = q / per_group, rem = q % per_group;
    t.nt = xcd * per_x + rem / inner_n;
    t.inner = rem % inner_n;
    t.live = slot < a.G;
    t.g = t.live ? (a.order ? a.order[slot] : slot) : 0;
    return t;
}
inline long long tile_grid_blocks(const WsGemmArgs& a, int n_tiles, int inner_n) {
    // (the spread mapping needs G * n_tiles * inner_n blocks, never more than the first case below)
    if (a.G >= kXcd) return (long long)(a.G + kXcd - 1) / kXcd * kXcd * n_tiles * inner_n;
    if (a.ksplit == 1 && inner_n >= kXcd) return (long long)a.G * ((inner_n + kXcd - 1) / kXcd) * n_tiles * kXcd;
    return ((long long)a.G * n_tiles + kXcd - 1) / kXcd * kXcd * inner_n;
}

// Of a grid sized for `most` inner tiles per (group, column tile): the virtual blocks that deal inner_n of them.  Exact where the K of a
// product is split (the grid then is a multiple of `most`); elsewhere the two are the same and so are the blocks.
__host__ __device__ __forceinline__ int blocks_dealt(int most_blocks, int most, int inner_n) {
    return inner_n == most ? most_blocks : most_blocks / most * inner_n;
}

// Top-1 combine fused into GEMM-2 leaves rows of dropped tokens unwritten: zero them (or copy what is added to), spread over the waves of all
// work-groups (a dropped token has no other writer).  A wave looks at 16 tokens at once: one token after the other, a
// work-group of a small grid waited for up to 16 memory round trips before its first tile (8192 tokens, 512 work-groups).
template <bool ADD = false> __device__ __forceinline__ void zero_dropped_rows(const WsGemmArgs& a, int tid, int nthreads) {
    if (!a.zero_slot_idx) return;
    for_dropped_tokens(a.zero_slot_idx, 1, a.T, tid, nthreads, [&](int t, int lane) {
        uint4* o = reinterpret_cast<uint4*>(a.out + (size_t)t * a.N);
        for (int i = lane; i < a.N / 8; i += kWave)
            o[i] = ADD && a.add ? reinterpret_cast<const uint4*>(a.add + (size_t)t * a.N)[i] : make_uint4(0, 0, 0, 0);
    });
}

// 16-byte loads and stores with the non-temporal hint: data that passes through once (expert weights at a
// few rows per expert, results nobody reads soon) should not push reusable lines out of the caches.
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_stream16(const void* p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_stream16(void* p, const uint4 o) {
    const u32x4_t v = {o.x, o.y, o.z, o.w};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(p));
}

// 8 bf16 biases of columns n_lane.. as loaded (zero without a bias vector), and their fp32 values
__device__ __forceinline__ uint4 load_bias_raw(const WsGemmArgs& a, int g, int n_lane) {
    return a.bias ? *reinterpret_cast<const uint4*>(a.bias + (size_t)g * a.N + n_lane) : make_uint4(0, 0, 0, 0);
}
__device__ __forceinline__ void unpack_bias8(const uint4 bv, float (&bias)[8]) {
    bias[0] = __uint_as_float(bv.x << 16); bias[1] = __uint_as_float(bv.x & 0xffff0000u);
    bias[2] = __uint_as_float(bv.y << 16); bias[3] = __uint_as_float(bv.y & 0xffff0000u);
    bias[4] = __uint_as_float(bv.z << 16); bias[5] = __uint_as_float(bv.z & 0xffff0000u);
    bias[6] = __uint_as_float(bv.w << 16); bias[7] = __uint_as_float(bv.w & 0xffff0000u);
}
__device__ __forceinline__ void load_bias8(const WsGemmArgs& a, int g, int n_lane, float (&bias)[8]) {
    unpack_bias8(load_bias_raw(a, g, n_lane), bias);
}

// NC (8, 4, 2 or 1) consecutive 16-bit values as one access
template <int NC> struct Bf16Vec;
template <> struct Bf16Vec<8> { typedef uint4 type; };
template <> struct Bf16Vec<4> { typedef uint2 type; };
template <> struct Bf16Vec<2> { typedef uint32_t type; };
template <> struct Bf16Vec<1> { typedef uint16_t type; };
__device__ __forceinline__ uint32_t raw_dword(const uint4& v, int q) { return dw(v, q); }
__device__ __forceinline__ uint32_t raw_dword(const uint2& v, int q) { return q == 0 ? v.x : v.y; }
__device__ __forceinline__ uint32_t raw_dword(const uint32_t& v, int) { return v; }
__device__ __forceinline__ uint32_t raw_dword(const uint16_t& v, int) { return v; }
// fp32 value i of NC loaded bf16 values
template <typename V> __device__ __forceinline__ float bf16_of(const V& v, int i) {
    const uint32_t d = raw_dword(v, i / 2);
    return __uint_as_float(i & 1 ? d & 0xffff0000u : d << 16);
}
template <int NC> __device__ __forceinline__ void load_bias(const WsGemmArgs& a, int g, int n, float (&bias)[NC]) {
    typename Bf16Vec<NC>::type v{};
    if (a.bias) v = *reinterpret_cast<const typename Bf16Vec<NC>::type*>(a.bias + (size_t)g * a.N + n);
#pragma unroll
    for (int i = 0; i < NC; ++i) bias[i] = bf16_of(v, i);
}

// Token and gate probability of expert row `row` of group g (top-1 combine fused into GEMM-2)
__device__ __forceinline__ void scatter_lookup(const WsGemmArgs& a, int g, int row, int& t, float& gw) {
    t = a.scatter_map[(size_t)g * a.scatter_stride + row];
    gw = a.gate_w[(size_t)t * a.top_k];
}

// Finishes NC (8, 4, 2 or 1) consecutive columns n_lane.. of row `row` (index inside group g): v = acc + bias on entry.
// EPI_SCATTER: (t, gw) = scatter_lookup of the row, fetched by the caller.  ADD: a.add is looked at (the kernels of a decode step; in
// the tiled ones its test alone cost 16384-wide products on plain weights 0.6 %).
template <int EPI, int NC = 8, bool ADD = false>
__device__ __forceinline__ void finish_row(const WsGemmArgs& a, int g, int row, int ks, int n_lane, float (&v)[NC],
                                           int t = 0, float gw = 1.f) {
    typedef typename Bf16Vec<NC>::type Vec;
    const long long grow = (long long)g * a.o_group_stride + row;   // row in [G, o_group_stride]
    if constexpr (EPI == EPI_PARTIAL) {
        static_assert(NC >= 4, "16-byte stores");
        float* o = a.partial + ((size_t)ks * a.partial_rows + grow) * a.N + n_lane;
#pragma unroll
        for (int q = 0; q < NC / 4; ++q)
            *reinterpret_cast<float4*>(o + 4 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        return;
    }
    size_t orow = (size_t)grow;
    if (EPI == EPI_GELU) {
#pragma unroll
        for (int i = 0; i < NC; ++i) v[i] = gelu_tanh(v[i]);
    } else if (EPI == EPI_SCATTER) {
#pragma unroll
        for (int i = 0; i < NC; ++i) v[i] *= gw;
        orow = (size_t)t;
    } else if (EPI == EPI_COMBINE) {
        // dense branch + sum_j keep_j g_j ye[e_j, slot_j, :] for token grow
        for (int j = 0; j < a.top_k; ++j) {
            const int s = a.slot_idx[grow * a.top_k + j];
            if (s < 0) continue;
            const int e = a.expert_idx[grow * a.top_k + j];
            const float gw = a.gate_w[grow * a.top_k + j];
            const uint16_t* yp = a.ye + ((size_t)e * a.C + s) * a.N + n_lane;
            const Vec y = *reinterpret_cast<const Vec*>(yp);
#pragma unroll
            for (int i = 0; i < NC; ++i) v[i] = fmaf(gw, bf16_of(y, i), v[i]);
        }
    }
    if constexpr (ADD && (EPI == EPI_SCATTER || EPI == EPI_COMBINE)) {
        if (a.add) {
            const Vec y = *reinterpret_cast<const Vec*>(a.add + orow * a.N + n_lane);
#pragma unroll
            for (int i = 0; i < NC; ++i) v[i] += bf16_of(y, i);
        }
    }
    uint32_t o[(NC + 1) / 2];
#pragma unroll
    for (int q = 0; q < (NC + 1) / 2; ++q) o[q] = pack_bf16x2(v[2 * q], NC > 1 ? v[(2 * q + 1) % NC] : 0.f);
    // h and the layer output are written once and read much later or never: streaming stores keep them
    // from displacing the activation rows in L2.  Expert outputs and split-K partials are read back at once.
    uint16_t* dst = a.out + orow * a.N + n_lane;
    if constexpr (NC == 8) {
        const uint4 ov = make_uint4(o[0], o[1], o[2], o[3]);
        if (EPI == EPI_STORE) *reinterpret_cast<uint4*>(dst) = ov;
        else store_stream16(dst, ov);
    } else if constexpr (NC == 4) {
        const uint2 ov = make_uint2(o[0], o[1]);
        if (EPI == EPI_STORE) *reinterpret_cast<uint2*>(dst) = ov;
        else __builtin_nontemporal_store(__builtin_bit_cast(unsigned long long, ov), reinterpret_cast<unsigned long long*>(dst));
    } else {                                                        // a piece of a line that other work-groups complete
        *reinterpret_cast<Vec*>(dst) = static_cast<Vec>(o[0]);
    }
}

}  // namespace moe
