// Tiled bf16 MFMA grouped GEMM on packed weights: 256-column tiles of 256 or 128 rows on four waves (ffn_tile.hip has the other
// shapes, the other weight layout and the choice of the shape).
//
// A work-group owns BM rows x 256 columns, each of its four waves every other 16-row sub-tile of 128 columns.  The
// accumulators of a full tile take 256 registers per lane (the accumulation half of the file), the operand fragments of two
// 32-deep steps the other half.  (The 256-row store and GELU instances have two or three values too many: written to scratch memory
// before the main loop and read back in the epilogue.)
//
// What bounds it: on random operands the chip runs at its power limit (1.8 - 2.0 GHz instead of 2.4), so bytes moved per flop
// count twice, as time and as clock.  128 x 128 per wave reads 64 KB of fragments from LDS per 32-deep step of a tile, eight
// waves of 64 x 128 read 96.  Activations come in chunks of 64 k: a load takes 128 bytes of a row, a whole cache line; 32-deep
// stages ask for every line twice (loads alone, 8192 x 4096 x 4096: 17.8 TB/s from L2 with 64-byte pieces, 23.2 with 128).  One
// barrier per 64 k.  Products alone, against the eight-wave kernel of 32-deep stages: 8192 x 4096 x 4096 204 -> 190 us (1.45
// PFLOP/s; two of them in moe_expert_ffn 435 -> 394), 8 x 2048 x 4096 x 1024 105 -> 96, 64 groups of 256 x 4096 x 1024 146 -> 131,
// with bias + GELU 32 groups of 256 x 1024 x 4096 79 -> 76; 128-row tiles: 64 x 128 x 1024 x 4096 with GELU 122 -> 116, 32 x 256 x
// 4096 x 1024 94 -> 79, 8 x 1024 x 4096 x 1024 63 -> 58.  Layers: 8192 tokens, 1024 / 4096, 32 experts beside a dense branch 314 ->
// 292 us, 64 experts 403 -> 377.
// With one wave per SIMD nothing covers a wave's own waits, so every load, LDS read and scalar instruction sits between two
// matrix instructions, and the epilogue's exp and rcp are taken eight at a time.
#pragma once

#include "ffn_common.h"
#include <type_traits>

namespace moe {

constexpr int kChunk = 64;                       // k per chunk of the ring: 128 bytes of an activation row
constexpr int kWideCols = 256, kWideThreads = 256;
constexpr int kWideB = kChunk * kWideCols * 2;   // weight bytes of a chunk
constexpr int kWideLds = 160 * 1024;

// Ring of a tile whose waves work on ACT sub-tiles each (32 ACT rows): NA activation and NB weight chunks.
template <int ACT> struct WideRing {
    static constexpr int A_BYTES = ACT * 32 * kChunk * 2;
    static constexpr int NA = ACT > 4 ? 2 : ACT > 2 ? 3 : 4;
    static constexpr int NB = ACT > 2 ? 3 : 4;
    static constexpr int B0 = NA * A_BYTES;
    static_assert(B0 + NB * kWideB <= kWideLds, "the ring must fit a compute unit's LDS");
    // loads of a wave that may be in flight when chunk c + 1 is needed, at the barrier in the middle of chunk c: those
    // issued after A(c + 1) and after B(c + 1)
    static constexpr int AFTER_A = 8 * (NA - 1) + ACT * (NA - 2), AFTER_B = (8 + ACT) * (NB - 2);
    static constexpr int ALLOWED = AFTER_A < AFTER_B ? AFTER_A : AFTER_B;
    static_assert(NA >= 2 && NB >= 3 && ALLOWED < 64, "vmcnt is a 6-bit counter");
};

__device__ __align__(16) const uint32_t kWideZero16[4] = {0, 0, 0, 0};   // what lanes past K load

// LDS address of the next direct loads; one wait state before the first of them
template <int IMM> __device__ __forceinline__ void set_m0(uint32_t base) {
    asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0" ::"s"(base), "n"(IMM) : "memory", "m0", "scc");
}
// 16 bytes per lane from global memory to LDS at m0 + OFF + 16 lane; OFF is added to the global address too.  NT: with the
// non-temporal hint
template <int OFF, bool NT> __device__ __forceinline__ void dma16_at(const uint16_t* g) {
    if (NT) asm volatile("global_load_lds_dwordx4 %0, off offset:%1 nt" ::"v"(g), "n"(OFF) : "memory");
    else asm volatile("global_load_lds_dwordx4 %0, off offset:%1" ::"v"(g), "n"(OFF) : "memory");
}
// Matrix instructions as inline asm: with 256 accumulator registers the compiler does not update them in place by itself.
// It does not see what the statement is and puts no wait states around it.  The ones that a vector instruction needs on an
// operand or a result (2 before, 11 after) cannot be missing as long as the compiler copies no accumulator between two
// statements: they get their first values by statements of their own, each loop's body ends in mfma_guard(), and
// tests/test_wide_hazards.py looks through the built code.
__device__ __forceinline__ void mfma(f32x4_t& d, const bf16x8_t& a, const bf16x8_t& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void set_acc(f32x4_t& d, float v) {
    float x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("v_accvgpr_write_b32 %0, %1" : "=a"(x[i]) : "v"(v));
    d = f32x4_t{x[0], x[1], x[2], x[3]};
}
__device__ __forceinline__ void mfma_guard() { asm volatile("s_nop 10" ::: "memory"); }
template <int N> __device__ __forceinline__ void wait_vmcnt_barrier() {      // and this wave's LDS reads are done
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// gelu_tanh of eight values, step by step for all of them: one after the other, each would wait for its own exp and rcp, with no
// second wave on the SIMD to fill the time
__device__ __forceinline__ void gelu_tanh8(float (&v)[8]) {
    float p[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = fmaf(v[j] * v[j], kGelu3, kGelu1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = __builtin_amdgcn_exp2f(v[j] * p[j]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = __builtin_amdgcn_rcpf(1.0f + p[j]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] *= p[j];
}

// How the weights are read: through the caches, with the non-temporal hint, or as each tile's group needs it.  The hint is for
// weights that one row tile reads and nobody will find in the 256 MB Infinity Cache later.
enum WidePolicy { WIDE_CACHED, WIDE_STREAMED, WIDE_BY_GROUP };
constexpr bool wide_hints(int epi) { return epi == EPI_STORE || epi == EPI_GELU || epi == EPI_SCATTER; }   // the epilogues that have the hint

template <int BM, int EPI, bool RAGGED, int POLICY>
__global__ __launch_bounds__(kWideThreads, 1) void wide_kernel(const WsGemmArgs a0, const WsGemmArgs a1, const int split) {
    const bool second = (int)blockIdx.x >= split;                // uniform over the work-group
    const WsGemmArgs& a = second ? a1 : a0;
    const int block = second ? (int)blockIdx.x - split : (int)blockIdx.x;

    extern __shared__ __attribute__((aligned(16))) char lds[];   // activation ring, then weight ring
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, kg = lane >> 4;
    const int wm = w >> 1, wn = w & 1;

    const int n_tiles = (a.N + kWideCols - 1) / kWideCols;
    const int m_tiles = (a.max_rows + BM - 1) / BM;
    const TileId tile = tile_spread(a, n_tiles) ? tile_of_block_spread(a, n_tiles, m_tiles, block)
                                                : tile_of_block(a, n_tiles, m_tiles, block);
    const int g = tile.g, nt = tile.nt, mt = tile.inner;

    if (EPI == EPI_SCATTER) zero_dropped_rows(a, tid, kWideThreads);
    if (!tile.live) return;
    const int rows = a.rows ? min(a.rows[g], a.max_rows) : a.fixed_rows;
    const int m0 = mt * BM;
    if (m0 >= rows) return;
    const int nrows = min(BM, rows - m0);

    auto run = [&](auto act_c, auto nt_c) {
        constexpr int ACT = decltype(act_c)::value;
        constexpr bool NT = decltype(nt_c)::value;
        typedef WideRing<ACT> R;
        constexpr int NA = R::NA, NB = R::NB;
        const int chunks = (a.K + kChunk - 1) / kChunk;
        const int n0 = nt * kWideCols;

        // ---- sources of the direct loads ---------------------------------------------------------------------
        // activations: wave w, load i copies 128 bytes of rows (w*ACT + i)*8 ..+7; lane -> row +lane/8, 16-byte slot lane%8,
        // which holds k-piece slot ^ (row/2 % 8).  The loads i..i+3 share one LDS base: load i adds 1 KB (i%4) to both
        // addresses, which the pointer takes back here.
        // All of a tile's table look-ups and its bias are asked for before the first is waited for: with the choice between
        // table and group inside the loop the compiler made each row's look-up a memory round trip of its own.
        const int n_lane = n0 + wn * 128 + c * 8;                // this lane's eight columns
        const bool has_bias = EPI != EPI_PARTIAL && a.bias != nullptr;
        const uint4 bias_raw = has_bias ? *reinterpret_cast<const uint4*>(a.bias + (size_t)g * a.N + min(n_lane, a.N - 8)) : make_uint4(0, 0, 0, 0);
        const uint16_t* a_src[ACT];
        const int a_piece = (lane & 7);
        int a_row[ACT];
#pragma unroll
        for (int i = 0; i < ACT; ++i) a_row[i] = m0 + min((w * ACT + i) * 8 + (lane >> 3), nrows - 1);   // rows past the end alias the last valid one
        if (a.row_map) {
            const int32_t* map = a.row_map + (size_t)g * a.map_stride;
#pragma unroll
            for (int i = 0; i < ACT; ++i) a_row[i] = map[a_row[i]];
        }
        const uint16_t* a_group = a.A + (a.row_map ? (size_t)0 : (size_t)g * a.a_group_stride * a.K);
#pragma unroll
        for (int i = 0; i < ACT; ++i) {
            const int rt = (w * ACT + i) * 8 + (lane >> 3);
            a_src[i] = a_group + (size_t)a_row[i] * a.K + (a_piece ^ ((rt >> 1) & 7)) * 8 - (i & 3) * 512;
        }
        // weights: wave w copies fragments 4w..4w+3 of the tile's sixteen in each of a chunk's two 32-deep steps
        const int p_ng = (a.N + 127) / 128, kb_n = (a.K + 31) / 32;
        const int p_grp = min(n0 / 128 + w / 2, p_ng - 1);       // clamped group: loaded, never stored
        const size_t b_step = (size_t)p_ng * 4096;               // elements from one 32-deep step to the next
        const uint16_t* b_src = a.B + ((size_t)g * kb_n * p_ng + p_grp) * 4096 + (w & 1) * 2048 + lane * 8;
        const uint32_t a_dst = __builtin_amdgcn_readfirstlane(lds0 + w * (ACT * 1024));
        const uint32_t b_dst = __builtin_amdgcn_readfirstlane(lds0 + R::B0 + w * 4096);
        const uint16_t* zeros = reinterpret_cast<const uint16_t*>(kWideZero16);

        // load i of the activation chunk at k0 into the slot at `slot` / of the weight chunk whose data start at bp
        auto load_a = [&](auto ic, uint32_t slot, int k0) {
            constexpr int i = decltype(ic)::value;
            if constexpr (i < ACT) {
                if constexpr (i % 4 == 0) set_m0<(i / 4) * 4096>(a_dst + slot);
                const uint16_t* p = a_src[i] + k0;
                if (RAGGED) {
                    const int rt = (w * ACT + i) * 8 + (lane >> 3);
                    if (k0 + (a_piece ^ ((rt >> 1) & 7)) * 8 >= a.K) p = zeros - (i & 3) * 512;
                }
                dma16_at<(i % 4) * 1024, false>(p);
            }
        };
        auto load_b = [&](auto ic, uint32_t slot, int chunk, const uint16_t* bp) {
            constexpr int i = decltype(ic)::value, half = i / 4;
            if constexpr (i % 4 == 0) set_m0<half * (kWideB / 2)>(b_dst + slot);
            const uint16_t* p = half ? bp + b_step : bp;
            if (RAGGED && half == 1 && 2 * chunk + 1 >= kb_n) p = zeros - (i & 3) * 512;
            dma16_at<(i % 4) * 1024, NT>(p);
        };
#define MOE_IC(i) std::integral_constant<int, i>()
#define MOE_EACH8(f) f(MOE_IC(0)); f(MOE_IC(1)); f(MOE_IC(2)); f(MOE_IC(3)); f(MOE_IC(4)); f(MOE_IC(5)); f(MOE_IC(6)); f(MOE_IC(7))
        auto fill_a = [&](uint32_t slot, int chunk) {
            auto one = [&](auto ic) { load_a(ic, slot, chunk * kChunk); };
            MOE_EACH8(one);
        };
        auto fill_b = [&](uint32_t slot, int chunk) {
            const uint16_t* bp = b_src + (size_t)(2 * chunk) * b_step;
            auto one = [&](auto ic) { load_b(ic, slot, chunk, bp); };
            MOE_EACH8(one);
        };


        float bias[8];
        unpack_bias8(bias_raw, bias);
#pragma unroll
        for (int j = 0; j < 8; ++j) asm volatile("" : "+v"(bias[j]));   // waited for here, not behind the direct loads
        f32x4_t acc[ACT][8];

        // fragments of one 32-deep step: activations of sub-tiles 2i + wm, weights of this wave's 128 columns
        struct Frags { bf16x8_t a[ACT], b[8]; };
        const int swz = (c >> 1) & 7;
        const int a_lane0 = wm * 2048 + c * 128 + ((kg ^ swz) * 16), a_lane1 = wm * 2048 + c * 128 + (((4 + kg) ^ swz) * 16);
        const int b_lane = R::B0 + wn * 8192 + lane * 16;
        auto read_frag = [&](Frags& f, int pa, int pb, int q) {  // the q-th of a step's reads
            if (q < ACT) f.a[q] = *reinterpret_cast<const bf16x8_t*>(lds + pa + q * 4096);
            else if (q < ACT + 8) f.b[q - ACT] = *reinterpret_cast<const bf16x8_t*>(lds + pb + (q - ACT) * 1024);
        };
        // One 32-deep step: the matrix instructions of `cur`; between them the next step's fragments are read and eight
        // direct loads issued (`dma`).
        constexpr int RPJ = (ACT + 8 + 5) / 6;                   // reads per column fragment: all in the first six of eight
        auto step = [&](const Frags& cur, Frags& nxt, int pa, int pb, auto dma) {
            auto column = [&](auto jc) {
                constexpr int j = decltype(jc)::value;
#pragma unroll
                for (int q = 0; q < RPJ; ++q) read_frag(nxt, pa, pb, j * RPJ + q);
                // the row sub-tiles back and forth: consecutive instructions share an operand
#pragma unroll
                for (int q = 0; q < ACT; ++q) {
                    const int i = j % 2 ? ACT - 1 - q : q;
                    if (q == ACT / 2) dma(jc);
                    mfma(acc[i][j], cur.a[i], cur.b[j]);
                }
            };
            MOE_EACH8(column);
        };

        // ---- main loop ---------------------------------------------------------------------------------------
        // Chunk ch: step 0 (its fragments are in f0) reads step 1's into f1 and fetches weight chunk ch + NB - 1 into the slot
        // that chunk ch - 1 left; then every wave has read all of chunk ch, and chunk ch + 1 has landed for all; step 1 reads
        // the first fragments of chunk ch + 1 and fetches activation chunk ch + NA into chunk ch's slot.
        // The waits count on every wave issuing ACT and 8 loads per chunk, in that order, and on loads completing in order.
        Frags f0, f1;
        uint32_t a_rd = 0, b_rd = 0, b_wr = (NB - 1) * kWideB;
        const int last = chunks - 1;
#pragma unroll
        for (int v = -4; v < 0; ++v) {                           // what the steps of chunks v = -4 .. -1 would have issued
            const int cb = v + NB - 1, ca = v + NA;
            if (cb >= 0) fill_b(cb * kWideB, min(cb, last));
            if (v == -1) {
                // the sums begin with the bias
#pragma unroll
                for (int i = 0; i < ACT; ++i)
#pragma unroll
                    for (int j = 0; j < 8; ++j) set_acc(acc[i][j], bias[j]);
                wait_vmcnt_barrier<R::ALLOWED>();
            }
            if (ca >= 0) fill_a(ca * R::A_BYTES, min(ca, last));
        }
#pragma unroll
        for (int q = 0; q < ACT + 8; ++q) read_frag(f0, a_lane0, b_lane, q);
        auto chunk_steps = [&](int ch, auto issue_c) {
            constexpr bool ISSUE = decltype(issue_c)::value;
            const uint32_t b_slot = b_wr, a_slot = a_rd;
            const uint16_t* b_next = b_src + (size_t)(2 * (ch + NB - 1)) * b_step;
            step(f0, f1, a_lane1 + a_rd, b_lane + b_rd + kWideB / 2, [&](auto jc) { if (ISSUE) load_b(jc, b_slot, ch + NB - 1, b_next); });
            b_wr = b_rd;
            b_rd = b_rd == (NB - 1) * kWideB ? 0 : b_rd + kWideB;
            a_rd = a_rd == (NA - 1) * R::A_BYTES ? 0 : a_rd + R::A_BYTES;
            wait_vmcnt_barrier<ISSUE ? R::ALLOWED : 0>();
            const int k_next = min(ch + NA, last) * kChunk;      // the activation ring may reach a chunk further than the weights'
            step(f1, f0, a_lane0 + a_rd, b_lane + b_rd, [&](auto jc) { if (ISSUE) load_a(jc, a_slot, k_next); });
            mfma_guard();
        };
        int ch = 0;
        for (; ch < chunks - (NB - 1); ++ch) chunk_steps(ch, std::true_type());
        for (; ch < chunks; ++ch) chunk_steps(ch, std::false_type());   // everything is on its way

        // ---- epilogue ----------------------------------------------------------------------------------------
        if (n_lane >= a.N) return;
        int kg_e = kg;
        asm volatile("" : "+v"(kg_e));                           // the address is formed here, not kept through the main loop
        // top-1 combine: tokens and gate weights of all the lane's rows in two round trips, not two for each row
        int tok[EPI == EPI_SCATTER ? ACT * 4 : 1];
        float gate[EPI == EPI_SCATTER ? ACT * 4 : 1];
        if constexpr (EPI == EPI_SCATTER) {
            const int32_t* map = a.scatter_map + (size_t)g * a.scatter_stride + m0;
#pragma unroll
            for (int q = 0; q < ACT * 4; ++q) tok[q] = map[min((2 * (q / 4) + wm) * 16 + kg_e * 4 + q % 4, nrows - 1)];
#pragma unroll
            for (int q = 0; q < ACT * 4; ++q) gate[q] = a.gate_w[(size_t)tok[q] * a.top_k];
        }
        uint16_t* dst = a.out + ((size_t)g * a.o_group_stride + m0 + wm * 16 + kg_e * 4) * a.N + n_lane;
#pragma unroll
        for (int i = 0; i < ACT; ++i) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int rl = (2 * i + wm) * 16 + kg * 4 + r;   // D: rows 4*(lane/16)+r, column lane%16
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = acc[i][j][r];
                if constexpr (EPI == EPI_STORE || EPI == EPI_GELU) {
                    if (EPI == EPI_GELU) gelu_tanh8(v);
                    if (rl < nrows) {
                        const uint4 o = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                                                   pack_bf16x2(v[6], v[7]));
                        if (EPI == EPI_STORE) *reinterpret_cast<uint4*>(dst) = o;
                        else store_stream16(dst, o);
                    }
                    dst += r < 3 ? (size_t)a.N : (size_t)a.N * 29;
                } else {
                    if (rl >= nrows) continue;
                    if constexpr (EPI == EPI_SCATTER) finish_row<EPI, 8>(a, g, m0 + rl, 0, n_lane, v, tok[4 * i + r], gate[4 * i + r]);
                    else finish_row<EPI, 8>(a, g, m0 + rl, 0, n_lane, v);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto run_rows = [&](auto nt_c) {
        if constexpr (BM > 128) {
            if (nrows > 192) return run(std::integral_constant<int, 8>(), nt_c);
            if (nrows > 128) return run(std::integral_constant<int, 6>(), nt_c);
        }
        if (nrows > 64) run(std::integral_constant<int, 4>(), nt_c);
        else if (nrows > 32) run(std::integral_constant<int, 2>(), nt_c);
        else run(std::integral_constant<int, 1>(), nt_c);
    };
    if constexpr (POLICY == WIDE_CACHED) run_rows(std::false_type());
    else if constexpr (POLICY == WIDE_STREAMED) run_rows(std::true_type());
    else if (a.stream && rows <= BM) run_rows(std::true_type());
    else run_rows(std::false_type());
}

template <int BM, int EPI, bool RAGGED, int POLICY> static int launch_wide_p(const WsGemmArgs& a, const WsGemmArgs* b, hipStream_t s) {
    const int n_tiles = (a.N + kWideCols - 1) / kWideCols;
    const long long blocks_a = tile_grid_blocks(a, n_tiles, (a.max_rows + BM - 1) / BM);
    const long long blocks_b = b ? tile_grid_blocks(*b, n_tiles, (b->max_rows + BM - 1) / BM) : 0;
    const long long blocks = blocks_a + blocks_b;                // both multiples of the XCD count
    if (blocks > (1ll << 30)) return MOE_ERR_UNSUPPORTED;        // block indices are ints in the kernel
    static OncePerDevice asked;
    const int rc = ask_lds(reinterpret_cast<const void*>(&wide_kernel<BM, EPI, RAGGED, POLICY>), kWideLds, asked);
    if (rc != MOE_OK) return rc;
    hipLaunchKernelGGL((wide_kernel<BM, EPI, RAGGED, POLICY>), dim3((unsigned)blocks), dim3(kWideThreads), kWideLds, s, a, b ? *b : a, (int)blocks_a);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}
template <int BM, int EPI, bool RAGGED> static int launch_wide_r(const WsGemmArgs& a, const WsGemmArgs* b, int policy, hipStream_t s) {
    if constexpr (wide_hints(EPI)) {
        if (policy == WIDE_STREAMED) return launch_wide_p<BM, EPI, RAGGED, WIDE_STREAMED>(a, b, s);
        if constexpr (BM == 256) {
            if (policy == WIDE_BY_GROUP) return launch_wide_p<BM, EPI, RAGGED, WIDE_BY_GROUP>(a, b, s);
        }
    }
    return launch_wide_p<BM, EPI, RAGGED, WIDE_CACHED>(a, b, s);
}
template <int EPI> int launch_wide_epi(const WsGemmArgs& a, const WsGemmArgs* b, int tile_rows, int policy, hipStream_t s) {
    if (tile_rows == 256)
        return a.K % kChunk ? launch_wide_r<256, EPI, true>(a, b, policy, s) : launch_wide_r<256, EPI, false>(a, b, policy, s);
    return a.K % kChunk ? launch_wide_r<128, EPI, true>(a, b, policy, s) : launch_wide_r<128, EPI, false>(a, b, policy, s);
}

}  // namespace moe
