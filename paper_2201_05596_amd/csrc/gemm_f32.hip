// Grouped GEMM of the fp32 layer on the fp32 matrix cores (paper Sec. 3.1: each expert is an FFN; this is one of its
// two products), with the layout transforms of Sec. 5.4 fused in as in the bf16 kernels:
//   out[g, r, n] = epi( sum_k A[row(g, r), k] B[g, k, n] + bias[g, n] ),  r < rows(g)
// where row() may go through the slot->token table (dispatch) and epi may scale by the gate probability and write the
// token's row, or add the expert outputs to the dense branch (combine).
//
// v_mfma_f32_16x16x4_f32, fp32 all the way.  A lane (c = lane % 16, kg = lane / 16) holds four consecutive k
// (4 kg .. 4 kg + 3 of a 16-deep block) of one activation row, and four consecutive columns 4c .. 4c + 3 of the weight
// rows with the same k: matrix instruction (j, i) multiplies element j of the first with element i of the second, so
// every operand is a 16-byte access, no value is moved between lanes, and a lane ends with four consecutive columns
// of four rows (16-byte stores).
//
// Two kernels:
//   * f32_tile_kernel, groups of more than 32 rows: bound by the fp32 matrix cores (157 TFLOP/s).  64 x 128 or
//     128 x 64 tiles of four 32 x 64 sub-tiles, each by two waves that halve every 32-deep chunk of K between them (one
//     work-group of eight waves has a compute unit to itself at the usual sizes, and one wave per SIMD left every LDS
//     and barrier wait exposed).  Chunks are double-buffered in LDS, fragments in registers; loads, LDS reads and LDS
//     writes of later chunks are placed between the matrix instructions of this one.  Weight rows of 256 bytes are read
//     without bank conflicts as they are; activation rows are padded to 160 bytes (2 x odd 16-byte units), which
//     sends the 16 lanes of one LDS pass (0-3, 12-15 of one kg, 4-11 of the next) to 16 different units.
//     1536 tokens, 512/2048, 8 experts, top-2 (12.9 GFLOP, 3.2 tiles per compute unit in GEMM-1, 0.8 in GEMM-2): 81 + 75 us
//     (83 TFLOP/s; 2048 matrix clocks of a chunk in about 2600).  Four waves with nothing placed: 88 + 101; on the
//     vector ALUs, before: 162 + 465.  One work-group per compute unit, by its 132 registers (within 128 two fit): with two, a
//     unit may hold two tiles while another has none, and a few rounds of tiles of unequal rows end later (layers, two / one: 1700
//     tokens, 1024/1024, 8 experts with room for 430 rows 156 / 97 us; 1919 tokens, 1024/2048, 4 experts with room for 720, skewed
//     185 / 160; 1000 tokens, 1024/4096, 16 experts, skewed 202 / 188).  Many full tiles would be a little faster with two (8192
//     tokens, 512/2048, 8 experts 294 / 303).
//   * f32_rows_kernel, groups of at most 32 rows (and, 32 rows at a time, products with few tiles and those of 2^24 columns or
//     more, whose 32-row chunks of weights are beyond the offsets of a buffer descriptor): a read of the weights, bound by latency
//     when they are few.  A work-group of eight waves owns 64 columns, the waves take 16-deep blocks of K in turn straight from
//     memory into registers, three blocks ahead, and add up through LDS in wave order.
//     256 tokens, 64/256, 8 experts: both products 48 us on the vector-ALU kernel before, 5.5 + 7.4 here.
#include <type_traits>

#include "moe_internal.h"

namespace moe {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Finishes columns n .. n + 3 of row r of group g (acc without the bias on entry).
template <int EPI>
__device__ __forceinline__ void f32_finish(const GemmArgs& a, int g, int r, int n, f32x4_t v) {
    const float* bias = static_cast<const float*>(a.bias);
    if (bias) v += *reinterpret_cast<const f32x4_t*>(bias + (size_t)g * a.N + n);
    size_t orow = (size_t)g * a.o_group_stride + r;
    if (EPI == EPI_GELU) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = gelu_tanh(v[i]);
    } else if (EPI == EPI_SCATTER) {
        orow = (size_t)a.scatter_map[(size_t)g * a.max_rows + r];
        v *= a.gate_w[orow * a.top_k];
    } else if (EPI == EPI_COMBINE) {
        for (int j = 0; j < a.top_k; ++j) {
            const int s = a.slot_idx[orow * a.top_k + j];
            if (s < 0) continue;
            const int e = a.expert_idx[orow * a.top_k + j];
            const float gw = a.gate_w[orow * a.top_k + j];
            const f32x4_t y = *reinterpret_cast<const f32x4_t*>(static_cast<const float*>(a.ye) + ((size_t)e * a.C + s) * a.N + n);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = fmaf(gw, y[i], v[i]);
        }
    }
    *reinterpret_cast<f32x4_t*>(static_cast<float*>(a.out) + orow * a.N + n) = v;
}

// EPI_SCATTER leaves the rows of dropped tokens unwritten: zero them, spread over all work-groups.
__device__ __forceinline__ void f32_zero_dropped(const GemmArgs& a, int tid, int nthreads) {
    for_dropped_tokens(a.slot_idx, a.top_k, a.T, tid, nthreads, [&](int t, int lane) {
        f32x4_t* o = reinterpret_cast<f32x4_t*>(static_cast<float*>(a.out) + (size_t)t * a.N);
        for (int i = lane; i < a.N / 4; i += kWave) o[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    });
}

__device__ __forceinline__ int f32_rows_of(const GemmArgs& a, int g) { return a.rows ? min(a.rows[g], a.max_rows) : a.fixed_rows; }
// activation row of (g, r)
__device__ __forceinline__ const float* f32_arow(const GemmArgs& a, int g, int r) {
    const long long ar = a.row_map ? (long long)a.row_map[(size_t)g * a.max_rows + r] : (long long)g * a.a_group_stride + r;
    return static_cast<const float*>(a.A) + (size_t)ar * a.K;
}

// ---- more than 32 rows per group -----------------------------------------------------------------------------
constexpr int kFK = 32;                       // k per chunk
constexpr int kFStride = kFK * 4 + 32;        // bytes per activation row in LDS

// WMW x WNW pairs of waves of 32 rows x 64 columns; wave 0 of a pair takes the first half of every chunk, wave 1 the second
template <int WMW, int WNW, int EPI>
__global__ __launch_bounds__(512, 2) void f32_tile_kernel(const GemmArgs a, const int n_tiles) {
    static_assert(WMW * WNW == 4, "four pairs of waves");
    constexpr int TM = WMW * 32, TN = WNW * 64;
    constexpr int A_BYTES = TM * kFStride, BUF = A_BYTES + kFK * TN * 4;
    constexpr int NPA = TM * kFK / 4 / 512, NPB = TN * kFK / 4 / 512;      // 16-byte pieces per thread and chunk
    __shared__ __attribute__((aligned(16))) char lds[2 * BUF];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, c = lane & 15, kg = lane >> 4;
    const int kh = w >> 2, wm = (w & 3) / WNW, wn = (w & 3) % WNW;
    if (EPI == EPI_SCATTER) f32_zero_dropped(a, tid, 512);
    // column tiles innermost: with a multiple of 8 of them all row tiles of a column tile run on one XCD and share its
    // weights in that L2, and every XCD has the same work however unevenly the rows fall on the groups
    const int nt = blockIdx.x % n_tiles, mt = blockIdx.x / n_tiles, g = blockIdx.y;
    const int rows = f32_rows_of(a, g), m0 = mt * TM, n0 = nt * TN;
    if (m0 >= rows) return;

    const float* a_src[NPA];
    int a_k[NPA];
    uint32_t a_dst[NPA];
#pragma unroll
    for (int i = 0; i < NPA; ++i) {
        const int p = tid + i * 512, r = p / (kFK / 4), kp = p % (kFK / 4);
        a_src[i] = f32_arow(a, g, min(m0 + r, rows - 1));                  // rows past the end repeat the last one
        a_k[i] = kp * 4;
        a_dst[i] = r * kFStride + kp * 16;
    }
    // Weight rows through a buffer descriptor that starts at the chunk: the lane's offsets never change, and rows past K
    // come back as zeros.
    const float* B = static_cast<const float*>(a.B) + (size_t)g * a.K * a.N;
    constexpr int B_STEP = 512 / (TN / 4);                                 // k-rows between two pieces of a thread
    const int b_off = (tid / (TN / 4) * a.N + min(n0 + tid % (TN / 4) * 4, a.N - 4)) * 4;   // columns past the end: never stored
    struct Chunk {
        f32x4_t a[NPA], b[NPB];
    };
    auto load = [&](Chunk& q, int k0) {
#pragma unroll
        for (int i = 0; i < NPA; ++i) q.a[i] = *reinterpret_cast<const f32x4_t*>(a_src[i] + min(k0 + a_k[i], a.K - 4));
        const int k_in = __builtin_amdgcn_readfirstlane(min(k0, a.K));
        const int left = __builtin_amdgcn_readfirstlane(min(a.K - k_in, kFK));       // rows of the chunk inside K
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(B + (size_t)k_in * a.N), 0, left * a.N * 4, 0x00027000);
#pragma unroll
        for (int i = 0; i < NPB; ++i)
            q.b[i] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, b_off + i * B_STEP * a.N * 4, 0, 0));
    };
    auto store = [&](const Chunk& q, int k0, int buf) {              // zeros past K (a multiple of 4: all four of a piece or none)
        char* base = lds + buf * BUF;
#pragma unroll
        for (int i = 0; i < NPA; ++i)
            *reinterpret_cast<f32x4_t*>(base + a_dst[i]) = k0 + a_k[i] < a.K ? q.a[i] : f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NPB; ++i) *reinterpret_cast<f32x4_t*>(base + A_BYTES + (tid + i * 512) * 16) = q.b[i];
    };

    const int chunks = (a.K + kFK - 1) / kFK;
    // The rest exists once per number MS of 16-row sub-tiles that a wave works on (sub-tiles past the last row are left
    // out; the choice is the wave's): branches inside one loop would move the accumulators around at every chunk.
    auto run = [&](auto ms_count) {
        constexpr int MS = decltype(ms_count)::value, NA = MS > 0 ? MS : 1;
        f32x4_t acc[NA][4];
#pragma unroll
        for (int ms = 0; ms < NA; ++ms)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[ms][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        struct Frags {
            f32x4_t a[NA], b[4];
        };
        auto read = [&](Frags& f, int buf) {
            if (MS == 0) return;
            const char* ap = lds + buf * BUF + (wm * 32 + c) * kFStride + kh * 64 + kg * 16;
            const char* bp = lds + buf * BUF + A_BYTES + ((kh * 16 + kg * 4) * TN + wn * 64 + c * 4) * 4;
#pragma unroll
            for (int ms = 0; ms < MS; ++ms) f.a[ms] = *reinterpret_cast<const f32x4_t*>(ap + ms * 16 * kFStride);
#pragma unroll
            for (int j = 0; j < 4; ++j) f.b[j] = *reinterpret_cast<const f32x4_t*>(bp + j * TN * 4);
        };
        auto multiply = [&](const Frags& f) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int ms = 0; ms < MS; ++ms)
                        acc[ms][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[ms][j], f.b[j][i], acc[ms][i], 0, 0, 0);
        };
        // In step ch the fragments of chunk ch are in registers and chunk ch + 1 is in LDS; its fragments are read while
        // ch is multiplied, ch + 2 goes from registers into the buffer that ch has left, ch + 3 is fetched.
        Chunk q0, q1;
        Frags f0, f1;
        load(q0, 0);
        load(q1, kFK);
        store(q0, 0, 0);
        load(q0, 2 * kFK);                               // past the end: in bounds (clamped), not used
        store(q1, kFK, 1);
        lds_barrier();
        read(f0, 0);
        auto step = [&](const Frags& cur, Frags& nxt, Chunk& ready, Chunk& refill, int ch) {
            lds_barrier();                               // ch + 1 is in LDS, and everybody has the fragments of ch
            read(nxt, (ch + 1) & 1);
            load(refill, (ch + 3) * kFK);
            multiply(cur);
            store(ready, (ch + 2) * kFK, ch & 1);
            // everything else goes into the shadow of the matrix instructions (32 clocks each)
            if (MS == 2) {
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);      // matrix
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);      // LDS read
                }
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);      // vector ALU
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);      // global load
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);      // LDS write
                    __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);           // nothing of the next step (a wait for its loads) moves up here
        };
        int ch = 0;
        for (; ch + 2 <= chunks; ch += 2) {
            step(f0, f1, q0, q1, ch);
            step(f1, f0, q1, q0, ch + 1);
        }
        if (ch < chunks) step(f0, f1, q0, q1, ch);
        lds_barrier();

        // the two halves of a pair's sums meet in LDS (the chunks' readers are done)
        f32x4_t* red = reinterpret_cast<f32x4_t*>(lds) + (w & 3) * 8 * 64 + lane;
        static_assert(4 * 8 * 64 * 16 <= 2 * BUF, "partial sums fit");
        if (kh == 1) {
#pragma unroll
            for (int q = 0; q < 4 * MS; ++q) red[q * 64] = acc[q / 4][q % 4];
        }
        lds_barrier();
        const int n = n0 + wn * 64 + c * 4;
        if (kh == 1 || n >= a.N) return;
#pragma unroll
        for (int q = 0; q < 4 * MS; ++q) acc[q / 4][q % 4] += red[q * 64];
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = m0 + wm * 32 + ms * 16 + kg * 4 + r;
                if (row < rows) f32_finish<EPI>(a, g, row, n, f32x4_t{acc[ms][0][r], acc[ms][1][r], acc[ms][2][r], acc[ms][3][r]});
            }
    };
    const int nsub = __builtin_amdgcn_readfirstlane(max(0, min(2, (rows - m0 - wm * 32 + 15) / 16)));
    if (nsub == 2) run(std::integral_constant<int, 2>());
    else if (nsub == 1) run(std::integral_constant<int, 1>());
    else run(std::integral_constant<int, 0>());
}

// ---- at most 32 rows per tile --------------------------------------------------------------------------------
constexpr int kFWaves = 8;                    // waves of a work-group = ways K is split
constexpr int kFAhead = 3;                    // 16-deep blocks in flight per wave

template <int MS, int EPI>
__global__ __launch_bounds__(kFWaves * 64, 4) void f32_rows_kernel(const GemmArgs a, const int n_tiles) {
    __shared__ __attribute__((aligned(16))) f32x4_t part[kFWaves][MS * 16][16];
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, kg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (EPI == EPI_SCATTER) f32_zero_dropped(a, tid, kFWaves * 64);
    const int nt = blockIdx.x % n_tiles, g = blockIdx.y;
    const int rows = f32_rows_of(a, g), m0 = blockIdx.x / n_tiles * MS * 16, n0 = nt * 64;
    if (m0 >= rows) return;

    const float* a_src[MS];
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) a_src[ms] = f32_arow(a, g, min(m0 + ms * 16 + c, rows - 1));
    const float* B = static_cast<const float*>(a.B) + (size_t)g * a.K * a.N + min(n0 + c * 4, a.N - 4);
    struct Block {
        f32x4_t av[MS], bv[4];
    };
    auto load = [&](Block& b, int kb) {
        const int k = kb * 16 + kg * 4;                      // K is a multiple of 4: a lane's four k are all inside or all outside
#pragma unroll
        for (int ms = 0; ms < MS; ++ms) b.av[ms] = *reinterpret_cast<const f32x4_t*>(a_src[ms] + min(k, a.K - 4));
#pragma unroll
        for (int j = 0; j < 4; ++j) b.bv[j] = *reinterpret_cast<const f32x4_t*>(B + (size_t)min(k + j, a.K - 1) * a.N);
    };
    f32x4_t acc[MS][4];
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[ms][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int blocks = (a.K + 15) / 16;
    const int mine = __builtin_amdgcn_readfirstlane(w < blocks ? (blocks - w + kFWaves - 1) / kFWaves : 0);   // blocks w, w + 8, ...
    auto multiply = [&](Block& b, int kb) {
        if (kb * 16 + 16 > a.K) {                            // K ends inside: zeros on both sides (0 times infinity is NaN)
            const bool in = kb * 16 + kg * 4 < a.K;
#pragma unroll
            for (int ms = 0; ms < MS; ++ms)
                if (!in) b.av[ms] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (!in) b.bv[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int ms = 0; ms < MS; ++ms)
                    acc[ms][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(b.av[ms][j], b.bv[j][i], acc[ms][i], 0, 0, 0);
    };
    Block st[kFAhead];
#pragma unroll
    for (int s = 0; s < kFAhead; ++s) load(st[s], w + s * kFWaves);        // past the end: in bounds (clamped), never multiplied
    int q = 0;
    for (; q + kFAhead <= mine; q += kFAhead) {
#pragma unroll
        for (int s = 0; s < kFAhead; ++s) {
            multiply(st[s], w + (q + s) * kFWaves);
            load(st[s], w + (q + s + kFAhead) * kFWaves);
            __builtin_amdgcn_sched_barrier(0);               // the refill stays here, kFAhead blocks ahead of its use
        }
    }
#pragma unroll
    for (int s = 0; s < kFAhead; ++s)
        if (q + s < mine) multiply(st[s], w + (q + s) * kFWaves);
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            part[w][ms * 16 + kg * 4 + r][c] = f32x4_t{acc[ms][0][r], acc[ms][1][r], acc[ms][2][r], acc[ms][3][r]};
    __syncthreads();
    const int row = tid / 16, n = n0 + (tid & 15) * 4;
    if (m0 + row >= rows || row >= MS * 16 || n >= a.N) return;
    f32x4_t v = part[0][row][tid & 15];
#pragma unroll
    for (int s = 1; s < kFWaves; ++s) v += part[s][row][tid & 15];
    f32_finish<EPI>(a, g, m0 + row, n, v);
}

template <int EPI> int launch_epi(const GemmArgs& a, hipStream_t s) {
    // groups along y: x alone is limited to 2^32 threads, which E * capacity reaches
    // Few tiles leave compute units idle, and the 32 x 64 ones of the rows kernel are four times as many.  They cost more per
    // flop, so the line is where two of them on every unit hold all (layers, us, second product on 64 x 128 / on 32 x 64: 1024
    // tokens, 512/2048, 8 experts, 256 small tiles 106 / 67; 300 tokens, 4 experts with a dense branch, both second products
    // 196 / 110; 2048 tokens, 8 experts, 512 tiles 124 / 105; 1536 tokens, top-2, 960 tiles 165 / 203.  First products: 700
    // tokens, 256/1024, 16 experts, 512 tiles 65.4 / 62.9; 512 tokens, 512/2048, 4 experts, 640 tiles 104 / 108).
    const long long small_tiles = ((long long)a.max_rows + 31) / 32 * (((long long)a.N + 63) / 64) * a.G;
    const bool few = a.max_rows <= 32 || small_tiles <= 512 || a.N >= 1 << 24;
    const bool narrow = a.N <= 64;                               // one 64-column tile: all four pairs along the rows
    const int tm = few ? (a.max_rows <= 16 ? 16 : 32) : narrow ? 128 : 64, tn = few || narrow ? 64 : 128;
    const int n_tiles = (int)(((long long)a.N + tn - 1) / tn);
    const long long tiles = ((long long)a.max_rows + tm - 1) / tm * n_tiles;
    if (tiles * 512 > 0xffffffffll) return MOE_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)tiles, (unsigned)a.G), block(512);
    static_assert(kFWaves * 64 == 512, "all kernels have the same work-group");
    if (few && tm == 16) hipLaunchKernelGGL((f32_rows_kernel<1, EPI>), grid, block, 0, s, a, n_tiles);
    else if (few) hipLaunchKernelGGL((f32_rows_kernel<2, EPI>), grid, block, 0, s, a, n_tiles);
    else if (narrow) hipLaunchKernelGGL((f32_tile_kernel<4, 1, EPI>), grid, block, 0, s, a, n_tiles);
    else hipLaunchKernelGGL((f32_tile_kernel<2, 2, EPI>), grid, block, 0, s, a, n_tiles);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

}  // namespace

int launch_gemm_f32(const GemmArgs& a, int epi, hipStream_t s) {
    if (a.max_rows <= 0 || a.G <= 0) return MOE_OK;
    if (a.K % 4 || a.N % 4) return MOE_ERR_INVALID_ARG;
    switch (epi) {
        case EPI_STORE: return launch_epi<EPI_STORE>(a, s);
        case EPI_GELU: return launch_epi<EPI_GELU>(a, s);
        case EPI_SCATTER: return launch_epi<EPI_SCATTER>(a, s);
        case EPI_COMBINE: return launch_epi<EPI_COMBINE>(a, s);
        default: return MOE_ERR_INVALID_ARG;
    }
}

}  // namespace moe
