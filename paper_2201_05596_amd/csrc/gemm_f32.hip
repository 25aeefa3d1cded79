// Grouped GEMM of the fp32 layer on the matrix cores (paper Sec. 3.1: each expert is an FFN; this is one of its
// two products), with the layout transforms of Sec. 5.4 fused in as in the bf16 kernels:
//   out[g, r, n] = epi( sum_k A[row(g, r), k] B[g, k, n] + bias[g, n] ),  r < rows(g)
// where row() may go through the slot->token table (dispatch) and epi may scale by the gate probability and write the
// token's row, or add the expert outputs to the dense branch (combine).
//
// v_mfma_f32_16x16x4_f32 (all but the split kernels): a lane (c = lane % 16, kg = lane / 16) holds four consecutive k
// (4 kg .. 4 kg + 3 of a 16-deep block) of one activation row, and four consecutive columns 4c .. 4c + 3 of the weight
// rows with the same k: matrix instruction (j, i) multiplies element j of the first with element i of the second, so
// every operand is a 16-byte access, no value is moved between lanes, and a lane ends with four consecutive columns
// of four rows (16-byte stores).
//
// Five kernels:
//   * f32_split_kernel, groups of more than 32 rows and K from 160 on (256 where its tiles are few): bound by the bf16 matrix cores and the
//     vector ALUs beside them.  An fp32 value is the exact sum of three bf16 ones, products of bf16 are exact in fp32, and six of the nine
//     products of pieces give an fp32 product at 2.6 times the fp32 matrix rate: the other three are 2^-27.5 of it (root mean square; 2^-24
//     at most).  64 x 128 tiles; sets of four waves of 64 x 32 split K, v_mfma_f32_32x32x16_bf16 (a matrix instruction keeps the vector
//     ALU from issuing for 8 clocks, so that six others fit beside one of 32 clocks, two beside one of 16 x 16 x 32).  Activations are
//     split once per tile and go through LDS, weights straight into the registers of the wave that multiplies them.
//     The instruction takes its 16 products in two groups of eight, one after the other: a group is cut to 2^-24 of its largest product,
//     its sum rounded into the accumulator.  So the product of two first pieces has accumulators of its own, which are rounded twice in 16 k
//     (the fp32 instructions round at every k), and the five small products theirs, whose roundings do not show.  In one accumulator, rounded
//     12 times in 16 k, sums of rectified values (zero products cost an fp32 chain no rounding) were up to 1.13 times as far from 64 bits as
//     fp32 ones.  Errors against 64 bits, fp32 / here with one set / with two: K = 512 3.3e-7 / 2.1e-7 / 1.8e-7, K = 2048 6.4e-7 / 3.5e-7 /
//     2.6e-7, operands of one sign 9.5e-8 / 9.2e-8 / 8.9e-8, rectified 4.2e-7 / 2.5e-7 / 1.9e-7, one column 1000 times the others 4.0e-7 / 2.8e-7
//     / 1.9e-7.
//     1536 tokens, 512/2048, 8 experts, top-2 (12.9 GFLOP): 81 + 75 us on f32_tile_kernel, 58 + 50 here; with both operands' pieces
//     through LDS 76 + 59 (every piece is written and read at half the rate it is used at).
//   * f32_tile_kernel, the same with shorter K or at most 64 columns: bound by the fp32 matrix cores (157 TFLOP/s).  64 x 128 or
//     128 x 64 tiles of four 32 x 64 sub-tiles, each by two waves that halve every 32-deep chunk of K between them (one
//     work-group of eight waves has a compute unit to itself at the usual sizes, and one wave per SIMD left every LDS
//     and barrier wait exposed).  Chunks are double-buffered in LDS, fragments in registers; loads, LDS reads and LDS
//     writes of later chunks are placed between the matrix instructions of this one.  Weight rows of 256 bytes are read
//     without bank conflicts as they are; activation rows are padded to 160 bytes (2 x odd 16-byte units), which
//     sends the 16 lanes of one LDS pass (0-3, 12-15 of one kg, 4-11 of the next) to 16 different units.
//     12.9 GFLOP in products of 512 x 2048 and 2048 x 512, 3.2 and 0.8 tiles per compute unit: 81 + 75 us (83 TFLOP/s; 2048
//     matrix clocks of a chunk in about 2600).  Four waves with nothing placed: 88 + 101; on the
//     vector ALUs, before: 162 + 465.  One work-group per compute unit, by its 132 registers (within 128 two fit): with two, a
//     unit may hold two tiles while another has none, and a few rounds of tiles of unequal rows end later (layers, two / one: 1700
//     tokens, 1024/1024, 8 experts with room for 430 rows 156 / 97 us; 1919 tokens, 1024/2048, 4 experts with room for 720, skewed
//     185 / 160; 1000 tokens, 1024/4096, 16 experts, skewed 202 / 188).  Many full tiles would be a little faster with two (8192
//     tokens, 512/2048, 8 experts 294 / 303).
//   * f32_ffn_kernel, d_model up to 64: both products in one launch;
//   * f32_rows_split_kernel, f32_rows_kernel's products of 17 rows and more with K from 512 on, on split operands;
//   * f32_rows_kernel, groups of at most 32 rows (and, 32 rows at a time, products with few tiles and those of 2^24 columns or
//     more, whose 32-row chunks of weights are beyond the offsets of a buffer descriptor): a read of the weights, bound by latency
//     when they are few.  A work-group of eight waves owns 64 columns, the waves take 16-deep blocks of K in turn straight from
//     memory into registers, three blocks ahead, and add up through LDS in wave order.
//     256 tokens, 64/256, 8 experts: both products 48 us on the vector-ALU kernel before, 5.5 + 7.4 here.
#include <type_traits>

#include "gate_common.h"
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

// ---- more than 32 rows per group, short K or few columns ------------------------------------------------------
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

// ---- more than 32 rows per group, long K: on the bf16 matrix instructions --------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
constexpr int kSRows = 64, kSCols = 128;      // of a tile: four waves of 32 columns

// Which elements of a vector of four sums the split does not hold (a bit each); they are taken again on the fp32 instructions.  bf16 ends
// at 2^-133, so up to 2^-134 of an operand is left out of its pieces.  With row and column the largest magnitudes in an element's row of
// activations and column of weights, K products lose less than K 2^-133 (row + column): 2^-25 of a sum of at least K 2^-108 (row + column).
// Smaller ones, zero included, are not held, unless the row or the column is all zeros.  Nor are sums that are not finite: pieces of
// infinities do not add up.
__device__ __forceinline__ int split_misses(const f32x4_t& v, int K, float row, const f32x4_t& column) {
    const float k = (float)K * 0x1p-108f;
    int bits = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bool small = fabsf(v[j]) < fmaf(k, column[j], k * row) && row != 0.f && column[j] != 0.f;
        bits |= (!(fabsf(v[j]) <= 3.4028234e38f) || small) << j;
    }
    return bits;
}

// the largest of a wave's values
__device__ __forceinline__ float wave_largest(float v) {
    v = fmaxf(v, dpp_f<kDppSwap1>(v));
    v = fmaxf(v, dpp_f<kDppSwap2>(v));
    v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
    v = fmaxf(v, dpp_f<kDppMirror>(v));                      // of 16 lanes
    const int b = __float_as_int(v);
    auto lane = [b](int l) { return __int_as_float(__builtin_amdgcn_readlane(b, l)); };
    return fmaxf(fmaxf(lane(0), lane(16)), fmaxf(lane(32), lane(48)));
}

// split_bf16x3 with the largest magnitude so far.  Infinities, NaN and values that round to infinity leave NaN in the later pieces.
template <int M> __device__ __forceinline__ void split_pairs(float (&x)[M][2], uint32_t (&piece)[3][M], float& largest) {
#pragma unroll
    for (int i = 0; i < M; ++i) largest = fmaxf(fmaxf(largest, fabsf(x[i][0])), fabsf(x[i][1]));
    split_bf16x3(x, piece);
}

// 16 rows x 64 columns from (m0, n0) on the fp32 matrix instructions, straight from memory: finishes the vectors of four sums that have bits in
// misses, taking the marked elements from here and the others from sums (both start at the rows and columns of this part of the tile).  So an
// element is the same whatever the other rows and columns hold.
template <int EPI>
__device__ void f32_unsplit(const GemmArgs& a, int g, int rows, int m0, int n0, int lane, const uint8_t* misses, const float* sums) {
    const int c = lane & 15, kg = lane >> 4, n = n0 + c * 4;
    uint32_t bits = 0;                                       // of the lane's four rows, a byte each
#pragma unroll
    for (int r = 0; r < 4; ++r) bits |= (uint32_t)misses[(kg * 4 + r) * (kSCols / 4) + c] << (8 * r);
    if (!__ballot(bits)) return;
    const float* A = f32_arow(a, g, min(m0 + c, rows - 1));
    const float* B = static_cast<const float*>(a.B) + (size_t)g * a.K * a.N + min(n, a.N - 4);
    f32x4_t acc[2][4] = {};                                  // every other 16 k: half as many steps that round a sum
    for (int k0 = 0; k0 < a.K; k0 += 32) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = k0 + h * 16 + kg * 4;              // K is a multiple of 4: a lane's four k are all inside or all outside
            f32x4_t av = {}, bv[4] = {};
            if (k < a.K) {
                av = *reinterpret_cast<const f32x4_t*>(A + k);
#pragma unroll
                for (int j = 0; j < 4; ++j) bv[j] = *reinterpret_cast<const f32x4_t*>(B + (size_t)(k + j) * a.N);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[h][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j], bv[j][i], acc[h][i], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[0][i] += acc[1][i];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int b = bits >> (8 * r) & 15;
        if (!b) continue;
        f32x4_t v = *reinterpret_cast<const f32x4_t*>(sums + (kg * 4 + r) * kSCols + c * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (b >> i & 1) v[i] = acc[0][i][r];
        f32_finish<EPI>(a, g, m0 + kg * 4 + r, n, v);
    }
}

// partial sums (less before), the largest values of rows and columns, flags, the largest values of waves, bits of split_misses
template <int P> constexpr int split_lds() { return P * kSRows * kSCols * 4 + (kSRows + kSCols + 4 + 8) * 4 + kSRows * kSCols / 4; }

// P sets of four waves split K between them, 32 deep in turn; wave 4 q + wn has columns 32 wn .. + 31 of the tile and set q's K.
template <int P, int EPI>
__global__ __launch_bounds__(P * 256, 2) void f32_split_kernel(const GemmArgs a, const int n_tiles) {
    constexpr int FRAG = 1024, PART = 2 * 2 * 3 * FRAG, BUF = P * PART, STEP = P * 32;      // STEP: k per step of the loop
    extern __shared__ __attribute__((aligned(16))) char lds[];
    static_assert(2 * BUF <= P * kSRows * kSCols * 4, "two buffers of activation pieces");
    float* const part = reinterpret_cast<float*>(lds);
    uint32_t* const largest = reinterpret_cast<uint32_t*>(lds + P * kSRows * kSCols * 4);        // [kSRows + kSCols], magnitudes as integers
    int* const flags = reinterpret_cast<int*>(largest + kSRows + kSCols);                        // [2]
    float* const wave_max = reinterpret_cast<float*>(flags + 4);                                 // [4 P]
    uint8_t* const misses = reinterpret_cast<uint8_t*>(wave_max + 8);                            // [kSRows][kSCols / 4]
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 31, half = lane >> 5;
    const int q = w >> 2, wn = w & 3;
    if (EPI == EPI_SCATTER) f32_zero_dropped(a, tid, P * 256);
    // column tiles innermost: with a multiple of 8 of them all row tiles of a column tile run on one XCD and share its
    // weights in that L2, and every XCD has the same work however unevenly the rows fall on the groups
    const int nt = blockIdx.x % n_tiles, mt = blockIdx.x / n_tiles, g = blockIdx.y;
    const int rows = f32_rows_of(a, g), m0 = mt * kSRows, n0 = nt * kSCols;
    if (m0 >= rows) return;
    if (tid < kSRows + kSCols + 2) largest[tid] = 0;             // and the flags

    // Activations: four threads take 32 k of a row, eight each, and put the pieces into LDS as fragments [row block][16 k][piece] of
    // v_mfma_f32_32x32x16_bf16.  Row r's 16 bytes of k-octet o stand at (o % 2) * 32 + (r ^ x(o)): x sends the lanes of one LDS
    // write to different banks.
    auto swizzle = [](int o) { return (o & 1) * 10 + (o >> 1) * 4; };
    const int oct = tid & 3, a_r = (tid & 255) >> 2;
    const float* const a_src = f32_arow(a, g, min(m0 + a_r, rows - 1));            // rows past the end repeat the last one
    char* const a_dst = lds + q * PART + ((a_r >> 5) * 6 + (oct >> 1) * 3) * FRAG + ((oct & 1) * 32 + ((a_r & 31) ^ swizzle(oct))) * 16;
    // values 4 h .. 4 h + 3 of a thread's eight of step t
    auto load_a = [&](f32x4_t& r, int h, int t) { r = *reinterpret_cast<const f32x4_t*>(a_src + min(t * STEP + q * 32 + oct * 8 + h * 4, a.K - 4)); };
    float row_max = 0.f, col_max = 0.f;                      // largest magnitudes that this thread splits
    // Every other set of waves sums the products negated: where a sum is cut to the grid of a larger product, the cut is not to nearest.
    const float sign = q % 2 ? -1.f : 1.f;
    uint32_t ua[3][4];                                       // pieces of a thread's eight values
    // Past K the weights are zeros, the activations any of the row's (an infinity there makes NaN, and those sums are taken again).
    auto split_a = [&](const f32x4_t& r, int h) {
        float x[2][2];
        uint32_t u[3][2];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j / 2][j % 2] = sign * r[j];
        split_pairs(x, u, row_max);
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 2; ++i) ua[p][2 * h + i] = u[p][i];
    };
    auto write_a = [&](int t) {
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(a_dst + (t & 1) * BUF + p * FRAG) = make_uint4(ua[p][0], ua[p][1], ua[p][2], ua[p][3]);
    };
    // Weights go straight into the registers of the wave that multiplies them: eight rows of a lane's column, through a buffer descriptor
    // that starts at the 16 rows of a half step (rows past K come back as zeros).
    const float* B = static_cast<const float*>(a.B) + (size_t)g * a.K * a.N;
    const int b_off = (half * 8 * a.N + min(n0 + wn * 32 + c, a.N - 1)) * 4;            // columns past the end: never stored
    // rows 4 h .. 4 h + 3 of a lane's eight in half step s of step t
    typedef uint32_t Pieces[3][4];
    auto load_b = [&](float (&r)[8], int h, int t, int s) {
        const int k_in = __builtin_amdgcn_readfirstlane(min(t * STEP + q * 32 + s * 16, a.K));
        const int left = __builtin_amdgcn_readfirstlane(min(a.K - k_in, 16));
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(B + (size_t)k_in * a.N), 0, left * a.N * 4, 0x00027000);
#pragma unroll
        for (int j = 4 * h; j < 4 * h + 4; ++j) r[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, b_off + j * a.N * 4, 0, 0));
    };
    auto split_b = [&](const float (&r)[8], int h, Pieces& f) {
        float x[2][2];
        uint32_t u[3][2];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j / 2][j % 2] = r[4 * h + j];
        split_pairs(x, u, col_max);
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 2; ++i) f[p][2 * h + i] = u[p][i];
    };

    const int steps = (a.K + STEP - 1) / STEP;
    // The loop exists once per number MS of row blocks that hold rows.
    auto run = [&](auto ms_count) {
        constexpr int MS = decltype(ms_count)::value;
        f32x16_t hi[MS], lo[MS];                             // sums of the products of two first pieces, and of the others
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int j = 0; j < 16; ++j) hi[ms][j] = lo[ms][j] = 0.f;
        auto read_a = [&](bf16x8_t (&f)[MS][3], int t, int s) {
            const char* p0 = lds + (t & 1) * BUF + q * PART + s * 3 * FRAG + (half * 32 + (c ^ swizzle(2 * s + half))) * 16;
#pragma unroll
            for (int ms = 0; ms < MS; ++ms)
#pragma unroll
                for (int p = 0; p < 3; ++p) f[ms][p] = *reinterpret_cast<const bf16x8_t*>(p0 + (ms * 6 + p) * FRAG);
        };
        // the six products of pieces that reach into the 24 bits of the sum
        auto multiply = [&](const bf16x8_t (&fa)[MS][3], const Pieces& fb, int from, int to) {
            constexpr int PA[6] = {0, 1, 2, 0, 1, 0}, PB[6] = {2, 1, 0, 1, 0, 0};
#pragma unroll
            for (int t = from; t < to; ++t)
#pragma unroll
                for (int ms = 0; ms < MS; ++ms) {
                    const uint32_t* f = fb[PB[t]];
                    f32x16_t& acc = t == 5 ? hi[ms] : lo[ms];
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ms][PA[t]], __builtin_bit_cast(bf16x8_t, make_uint4(f[0], f[1], f[2], f[3])), acc, 0, 0, 0);
                }
        };
        // Everything else goes into the shadow of the matrix instructions (32 clocks each, 24 of them free for six others), evenly: the
        // waves of a SIMD go through a step together.  A third TH of half step S each time.  Loads come when what they overwrite has been
        // split: any earlier they would get registers of their own, and copies.
        auto place = [&](auto s, auto third) {
            constexpr int S = decltype(s)::value, TH = decltype(third)::value;
            if (MS == 2) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                   // matrix
                    if (TH == 0) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                      // LDS read
                    if (TH == 0 && i < 2) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    if (TH != 1 || i == 1) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);            // global load
                    __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);                                   // vector ALU
                    if (S == 0 && TH == 0 && i > 0) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // LDS write
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        constexpr std::integral_constant<int, 0> c0;
        constexpr std::integral_constant<int, 1> c1;
        constexpr std::integral_constant<int, 2> c2;
        // Step t enters with its first half's fragments in registers, t's activations in LDS and half of t + 1's pieces in registers; what
        // is fetched is used a step later.
        float b0[8], b1[8];
        f32x4_t ra[2], first[2];
        bf16x8_t fa0[MS][3], fa1[MS][3];
        Pieces fb0, fb1;
        // (issued in the loop's order: the loop waits for all but so many)
        load_a(first[0], 0, 0);
        load_a(first[1], 1, 0);
        load_b(b0, 0, 0, 0);
        load_b(b0, 1, 0, 0);
        load_a(ra[0], 0, 1);
        split_a(first[0], 0);
        split_a(first[1], 1);
        write_a(0);
        split_b(b0, 0, fb0);
        split_b(b0, 1, fb0);
        split_a(ra[0], 0);
        __builtin_amdgcn_sched_barrier(0);
        load_a(ra[1], 1, 1);
        load_b(b1, 0, 0, 1);
        load_b(b1, 1, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        load_a(ra[0], 0, 2);
        load_b(b0, 0, 1, 0);
        lds_barrier();
        read_a(fa0, 0, 0);
        for (int t = 0; t < steps; ++t) {
            multiply(fa0, fb0, 0, 2);
            read_a(fa1, t, 1);
            load_b(b0, 1, t + 1, 0);
            split_a(ra[1], 1);
            write_a(t + 1);
            place(c0, c0);
            multiply(fa0, fb0, 2, 4);
            load_a(ra[1], 1, t + 2);
            split_b(b1, 0, fb1);
            place(c0, c1);
            multiply(fa0, fb0, 4, 6);
            load_b(b1, 0, t + 1, 1);
            split_b(b1, 1, fb1);
            place(c0, c2);
            lds_barrier();                               // t + 1 is in LDS, and everybody has the fragments of t
            multiply(fa1, fb1, 0, 2);
            read_a(fa0, t + 1, 0);
            load_b(b1, 1, t + 1, 1);
            split_a(ra[0], 0);
            place(c1, c0);
            multiply(fa1, fb1, 2, 4);
            load_a(ra[0], 0, t + 3);
            split_b(b0, 0, fb0);
            place(c1, c1);
            multiply(fa1, fb1, 4, 6);
            load_b(b0, 0, t + 2, 0);
            split_b(b0, 1, fb0);
            place(c1, c2);
        }

        // the sets' sums meet in LDS, in the order of the sets
        lds_barrier();
        const float in_wave = wave_largest(fmaxf(row_max, col_max));
        if (lane == 0) wave_max[w] = in_wave;
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int r = ms * 32 + 8 * (j / 4) + 4 * half + j % 4;                  // D: that row, column lane % 32
                part[((size_t)q * kSRows + r) * kSCols + wn * 32 + c] = hi[ms][j] + lo[ms][j];
            }
        lds_barrier();
        constexpr int NV = MS * 32 * kSCols / 4 / (P * 256);
        f32x4_t v[NV];
        float tile_max = wave_max[0];
#pragma unroll
        for (int s = 1; s < 4 * P; ++s) tile_max = fmaxf(tile_max, wave_max[s]);
        const f32x4_t columns_max = {tile_max, tile_max, tile_max, tile_max};
        int any = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int r = (tid + i * P * 256) / (kSCols / 4), n = tid % (kSCols / 4) * 4;
            v[i] = *reinterpret_cast<const f32x4_t*>(part + (size_t)r * kSCols + n);
#pragma unroll
            for (int p = 1; p < P; ++p) {
                const f32x4_t u = *reinterpret_cast<const f32x4_t*>(part + ((size_t)p * kSRows + r) * kSCols + n);
                v[i] = p % 2 ? v[i] - u : v[i] + u;
            }
            if (m0 + r < rows && n0 + n < a.N) any |= split_misses(v[i], a.K, tile_max, columns_max);
        }
        // Sums that are too small under the largest values of the whole tile are looked at again under those of their row and column.
        if (__ballot(any)) flags[0] = 1;
        lds_barrier();
        const bool again = flags[0];                         // uniform over the work-group
        int bits[NV] = {};
        if (again) {
            atomicMax(&largest[a_r], __float_as_uint(row_max));
            atomicMax(&largest[kSRows + wn * 32 + c], __float_as_uint(col_max));
            lds_barrier();
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int r = (tid + i * P * 256) / (kSCols / 4), n = tid % (kSCols / 4) * 4;
                if (m0 + r < rows && n0 + n < a.N)
                    bits[i] = split_misses(v[i], a.K, __uint_as_float(largest[r]), *reinterpret_cast<const f32x4_t*>(largest + kSRows + n));
                misses[r * (kSCols / 4) + n / 4] = bits[i];
                if (bits[i]) *reinterpret_cast<f32x4_t*>(part + (size_t)r * kSCols + n) = v[i];  // where this thread alone read before
            }
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int r = (tid + i * P * 256) / (kSCols / 4), n = n0 + tid % (kSCols / 4) * 4;
            if (m0 + r < rows && n < a.N && !bits[i]) f32_finish<EPI>(a, g, m0 + r, n, v[i]);
        }
        if (!again) return;
        lds_barrier();
        for (int i = w; i < 4 * MS; i += P * 4) {            // 16 rows x 64 columns at a time
            const int r = (i >> 1) * 16, n = (i & 1) * 64;
            f32_unsplit<EPI>(a, g, rows, m0 + r, n0 + n, lane, misses + r * (kSCols / 4) + n / 4, part + (size_t)r * kSCols + n);
        }
    };
    if (rows - m0 > 32) run(std::integral_constant<int, 2>());
    else run(std::integral_constant<int, 1>());
}

template <int P, int EPI> int launch_split(const GemmArgs& a, const dim3& grid, int n_tiles, hipStream_t s) {
    static OncePerDevice asked;
    const int rc = ask_lds(reinterpret_cast<const void*>(&f32_split_kernel<P, EPI>), split_lds<P>(), asked);
    if (rc != MOE_OK) return rc;
    hipLaunchKernelGGL((f32_split_kernel<P, EPI>), grid, dim3(P * 256), split_lds<P>(), s, a, n_tiles);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// ---- at most 32 rows per tile --------------------------------------------------------------------------------
constexpr int kFWaves = 8;                    // waves of a work-group = ways K is split
constexpr int kFAhead = 3;                    // 16-deep blocks in flight per wave

// sums of MS * 16 rows x 64 columns from (m0, n0) by W waves, a part by each: part is [W][MS * 16][16] in LDS.
// Eight sums whatever W is, each in a chain over every eighth block.
template <int MS, int W>
__device__ __forceinline__ void f32_rows_parts(const GemmArgs& a, f32x4_t* const part, int g, int rows, int m0, int n0) {
    constexpr int CHAINS = kFWaves / W, AHEAD = W == kFWaves ? kFAhead : CHAINS;
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, kg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
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
    f32x4_t acc[CHAINS][MS][4] = {};
    const int blocks = (a.K + 15) / 16;
    const int mine = __builtin_amdgcn_readfirstlane(w < blocks ? (blocks - w + W - 1) / W : 0);   // blocks w, w + 8, ...
    auto multiply = [&](Block& b, int kb, int chain) {
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
                    acc[chain][ms][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(b.av[ms][j], b.bv[j][i], acc[chain][ms][i], 0, 0, 0);
    };
    Block st[AHEAD];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) load(st[s], w + s * W);        // past the end: in bounds (clamped), never multiplied
    int q = 0;
    for (; q + AHEAD < mine; q += AHEAD) {               // the last round fetches nothing
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            multiply(st[s], w + (q + s) * W, s % CHAINS);
            load(st[s], w + (q + s + AHEAD) * W);
            __builtin_amdgcn_sched_barrier(0);               // the refill stays here, AHEAD blocks ahead of its use
        }
    }
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
        if (q + s < mine) multiply(st[s], w + (q + s) * W, s % CHAINS);
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) {
#pragma unroll
        for (int h = 1; h < CHAINS; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[0][ms][i] += acc[h][ms][i];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            part[(w * MS * 16 + ms * 16 + kg * 4 + r) * 16 + c] = f32x4_t{acc[0][ms][0][r], acc[0][ms][1][r], acc[0][ms][2][r], acc[0][ms][3][r]};
    }
    __syncthreads();
}
// columns 4 n .. 4 n + 3 of a row of the tile
template <int MS, int W> __device__ __forceinline__ f32x4_t f32_rows_sum(const f32x4_t* part, int row, int n) {
    f32x4_t v = part[row * 16 + n];
#pragma unroll
    for (int s = 1; s < W; ++s) v += part[(s * MS * 16 + row) * 16 + n];
    return v;
}

template <int MS, int EPI>
__global__ __launch_bounds__(kFWaves * 64, 4) void f32_rows_kernel(const GemmArgs a, const int n_tiles) {
    __shared__ __attribute__((aligned(16))) f32x4_t part[kFWaves * MS * 16 * 16];
    if (EPI == EPI_SCATTER) f32_zero_dropped(a, threadIdx.x, kFWaves * 64);
    const int nt = blockIdx.x % n_tiles, m0 = __builtin_amdgcn_readfirstlane(blockIdx.x / n_tiles * MS * 16), g = blockIdx.y;
    const int rows = f32_rows_of(a, g);
    if (m0 >= rows) return;
    f32_rows_parts<MS, kFWaves>(a, part, g, rows, m0, nt * 64);
    const int row = threadIdx.x / 16, n = nt * 64 + (threadIdx.x & 15) * 4;
    if (m0 + row >= rows || row >= MS * 16 || n >= a.N) return;
    f32_finish<EPI>(a, g, m0 + row, n, f32_rows_sum<MS, kFWaves>(part, row, threadIdx.x & 15));
}

// The same with 32 rows and K from 512 on on the bf16 matrix instructions, operands split as in f32_split_kernel: every wave splits what
// it loads, nothing is shared.  W waves share K: eight, which have a compute unit to themselves (few tiles then spread over the chip),
// or four, of which two or three work-groups share a unit.  Products, us, fp32 / eight waves / four: 4 x 75 rows, 2048 x 512 24.4 / 19.1
// / 19.3, 512 x 2048 17.9 / 15.2 / 13.9; 8 x 256, 2048 x 512 51.9 / 38.4 / 37.2, half of the tiles empty 50.2 / 20.8 / 33.7; 31 x 24, 512 x 2048 31.8 /
// 31.1 / 25.2; 1 x 60, 2048 x 512 24.0 / 18.6 / 19.4; 8 x 130, 800 x 200 12.4 / 10.2 / 10.4; 16 x 100, 256 x 1024 17.9 / 18.7 / 15.8.
// Errors against 64 bits 0.5 to 1.0 of the fp32 ones on every class of operands named at f32_split_kernel.  Not with a shorter K: there one
// large column among values of one sign, whose group's products are cut to its grid, is 1.02 .. 1.4 times as far off (K = 320 / 256 / 132: the
// fp32 sums are eight chains of few roundings), and there is little to gain.
template <int W> constexpr int rows_split_lds() { return W * 32 * 64 * 4 + (32 + 64 + 4 + W) * 4; }     // partial sums, largest values, flags
template <int W, int EPI>
__global__ __launch_bounds__(W * 64, 2) void f32_rows_split_kernel(const GemmArgs a, const int n_tiles) {
    constexpr int AHEAD = 2;                                     // 16-deep blocks in flight per wave
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float* const part = reinterpret_cast<float*>(lds);           // [W][32][64]
    uint32_t* const largest = reinterpret_cast<uint32_t*>(lds + W * 32 * 64 * 4);  // [32 rows + 64 columns], magnitudes as integers
    int* const flags = reinterpret_cast<int*>(largest + 32 + 64);                  // [2]
    float* const wave_max = reinterpret_cast<float*>(flags + 4);                   // [W]
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 31, half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (EPI == EPI_SCATTER) f32_zero_dropped(a, tid, W * 64);
    const int nt = blockIdx.x % n_tiles, m0 = __builtin_amdgcn_readfirstlane(blockIdx.x / n_tiles * 32), g = blockIdx.y;
    const int rows = f32_rows_of(a, g), n0 = nt * 64;
    if (m0 >= rows) return;
    if (tid < 32 + 64 + 2) largest[tid] = 0;                     // and the flags
    const float* const a_src = f32_arow(a, g, min(m0 + c, rows - 1));              // rows past the end repeat the last one
    const float* B = static_cast<const float*>(a.B) + (size_t)g * a.K * a.N;
    const int b_off = (half * 8 * a.N + min(n0 + c * 2, a.N - 2)) * 4;             // columns past the end: never stored
    const float sign = w % 2 ? -1.f : 1.f;                       // every other wave's sums negated, as in f32_split_kernel
    float row_max = 0.f, col_max[2] = {0.f, 0.f};
    struct Block {
        f32x4_t av[2];
        float bv[8][2];
    };
    const int blocks = (a.K + 15) / 16;
    const int mine = __builtin_amdgcn_readfirstlane(w < blocks ? (blocks - w + W - 1) / W : 0);   // blocks w, w + W, ...
    auto load = [&](Block& b, int i) {                           // past K: weights zero (also past the wave's last block), activations any
        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
        const int k_in = __builtin_amdgcn_readfirstlane(min((w + i * W) * 16, a.K));
        const int left = __builtin_amdgcn_readfirstlane(min(a.K - k_in, 16));
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(B + (size_t)k_in * a.N), 0, left * a.N * 4, 0x00027000);
#pragma unroll
        for (int h = 0; h < 2; ++h) b.av[h] = *reinterpret_cast<const f32x4_t*>(a_src + min(k_in + half * 8 + h * 4, a.K - 4));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const u32x2_t v = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(rs, b_off + j * a.N * 4, 0, 0));
            b.bv[j][0] = __uint_as_float(v[0]);
            b.bv[j][1] = __uint_as_float(v[1]);
        }
    };
    f32x16_t hi[2], lo[2];                                       // sums of the products of two first pieces, and of the others
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) hi[i][j] = lo[i][j] = 0.f;
    auto frag = [](const uint32_t (&u)[4]) { return __builtin_bit_cast(bf16x8_t, make_uint4(u[0], u[1], u[2], u[3])); };
    auto multiply = [&](const Block& b) {
        constexpr int PA[6] = {0, 1, 2, 0, 1, 0}, PB[6] = {2, 1, 0, 1, 0, 0};
        uint32_t ua[3][4], ub[2][3][4];
        float x[4][2];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j / 2][j % 2] = sign * b.av[j / 4][j % 4];
        split_pairs(x, ua, row_max);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j / 2][j % 2] = b.bv[j][i];
            split_pairs(x, ub[i], col_max[i]);
        }
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                f32x16_t& acc = t == 5 ? hi[i] : lo[i];
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(ua[PA[t]]), frag(ub[i][PB[t]]), acc, 0, 0, 0);
            }
    };
    Block st[AHEAD];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) load(st[s], s);
    int i = 0;
    for (; i + AHEAD < mine; i += AHEAD) {                       // the last round fetches nothing
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) {
            multiply(st[s]);
            __builtin_amdgcn_sched_barrier(0);
            load(st[s], i + s + AHEAD);
            __builtin_amdgcn_sched_barrier(0);                   // the refill stays here, AHEAD blocks ahead of its use
        }
    }
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
        if (i + s < mine) multiply(st[s]);
#pragma unroll
    for (int j = 0; j < 16; ++j)                                 // D: rows 8 (j / 4) + 4 half + j % 4, column lane % 32
        *reinterpret_cast<float2*>(part + (w * 32 + 8 * (j / 4) + 4 * half + j % 4) * 64 + c * 2) = make_float2(hi[0][j] + lo[0][j], hi[1][j] + lo[1][j]);
    const float lane_max = fmaxf(row_max, fmaxf(col_max[0], col_max[1])), in_wave = wave_largest(lane_max);
    if (lane == 0) wave_max[w] = in_wave;
    lds_barrier();
    constexpr int NV = 32 * 16 / (W * 64);
    const int n = (tid & 15) * 4;
    f32x4_t v[NV];
    float tile_max = wave_max[0];
#pragma unroll
    for (int s = 1; s < W; ++s) tile_max = fmaxf(tile_max, wave_max[s]);
    int any = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int row = tid / 16 + i * W * 4;
        v[i] = *reinterpret_cast<const f32x4_t*>(part + row * 64 + n);
#pragma unroll
        for (int s = 1; s < W; ++s) {
            const f32x4_t u = *reinterpret_cast<const f32x4_t*>(part + (s * 32 + row) * 64 + n);
            v[i] = s % 2 ? v[i] - u : v[i] + u;
        }
        if (m0 + row < rows && n0 + n < a.N) any |= split_misses(v[i], a.K, tile_max, f32x4_t{tile_max, tile_max, tile_max, tile_max});
    }
    // Sums that are too small under the largest values of the whole tile are looked at again under those of their row and column.
    if (__ballot(any)) flags[0] = 1;
    lds_barrier();
    if (flags[0]) {                                              // uniform over the work-group
        atomicMax(&largest[c], __float_as_uint(row_max));
#pragma unroll
        for (int i = 0; i < 2; ++i) atomicMax(&largest[32 + c * 2 + i], __float_as_uint(col_max[i]));
        lds_barrier();
        int bits[NV];
        any = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int row = tid / 16 + i * W * 4;
            const bool in = m0 + row < rows && n0 + n < a.N;
            bits[i] = in ? split_misses(v[i], a.K, __uint_as_float(largest[row]), *reinterpret_cast<const f32x4_t*>(largest + 32 + n)) : 0;
            any |= bits[i];
        }
        if (__ballot(any)) flags[1] = 1;
        lds_barrier();
        if (flags[1]) {                                          // marked elements from the fp32 instructions
            f32_rows_parts<2, W>(a, reinterpret_cast<f32x4_t*>(lds), g, rows, m0, n0);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const f32x4_t u = f32_rows_sum<2, W>(reinterpret_cast<f32x4_t*>(lds), tid / 16 + i * W * 4, tid & 15);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (bits[i] >> j & 1) v[i][j] = u[j];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int row = tid / 16 + i * W * 4;
        if (m0 + row < rows && n0 + n < a.N) f32_finish<EPI>(a, g, m0 + row, n0 + n, v[i]);
    }
}

// ---- both products of a narrow FFN -------------------------------------------------------------------------
// d_model up to 64, d_ffn up to 256: a work-group owns 16 MS rows and does both products; the intermediate never leaves its wave.  Wave w
// computes columns 32 w .. + 31 of the first product, two per lane, and they are just the K that it multiplies in the second: the
// rows turn from one operand order into the other through a piece of LDS of its own, no barrier until the waves' sums meet.  All
// weights are asked for before the first is used.  Bound by latency with few rows, by the fp32 matrix cores with many.  Sums are of 16 products,
// added afterwards: with chains of 32 in the second product the error against 64 bits is 1.05 .. 1.38 times that of two launches (64/64, one-sided
// operands 5.7e-8 / 7.5e-8), so 0.80 .. 1.00 (5.5e-8); the time is the same.
template <int MS, int EPI>
__global__ __launch_bounds__(kFWaves * 64, 2) void f32_ffn_kernel(const GemmArgs a, const GemmArgs b) {
    constexpr int HS = 36;                                       // floats per row of a wave's piece: 16 rows, 16 different units
    __shared__ __attribute__((aligned(16))) f32x4_t part[kFWaves][MS * 16][16];
    static_assert(HS * 4 <= 16 * 16, "a wave's rows of 32 columns fit where its sums go");
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, kg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto zero_dropped = [&]() {                                  // a memory round trip: behind the operands' loads, not before them
        __builtin_amdgcn_sched_barrier(0);
        if (EPI == EPI_SCATTER) f32_zero_dropped(b, tid, kFWaves * 64);
    };
    const int g = blockIdx.y, rows = f32_rows_of(a, g), m0 = blockIdx.x * MS * 16;
    if (m0 >= rows) return zero_dropped();
    const int d = a.K, f = a.N;
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    typedef float f32x2_t __attribute__((ext_vector_type(2)));

    f32x4_t x[4][MS];                                            // K of the first product: 16 deep blocks, zeros past it on both sides
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) {
        const float* src = f32_arow(a, g, min(m0 + ms * 16 + c, rows - 1));        // rows past the end repeat the last one
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4_t v = *reinterpret_cast<const f32x4_t*>(src + min(q * 16 + kg * 4, d - 4));
            x[q][ms] = q * 16 + kg * 4 < d ? v : zero;
        }
    }
    const float* W1 = static_cast<const float*>(a.B) + (size_t)g * d * f;
    const float* W2 = static_cast<const float*>(b.B) + (size_t)g * f * d + min(c * 4, d - 4);
    const float* bias1 = static_cast<const float*>(a.bias);
    float* const hs = reinterpret_cast<float*>(&part[w][0][0]);
    f32x4_t acc[2][MS][4];                                       // every 16 k of the second product on their own, too
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[0][ms][i] = acc[1][ms][i] = zero;
    const int n0 = w * 32;                                       // ffn_f32_fused: f is at most 8 x 32
    if (n0 < f) {
        const int n = n0 + c * 2, nc = min(n, f - 2);            // f is a multiple of 4: both columns inside or both outside
        f32x2_t w1[4][4], bv = {0.f, 0.f};
        f32x4_t w2[2][4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = q * 16 + kg * 4;
                const f32x2_t v = *reinterpret_cast<const f32x2_t*>(W1 + (size_t)min(k + j, d - 1) * f + nc);
                w1[q][j] = k < d ? v : f32x2_t{0.f, 0.f};
            }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = n0 + q * 16 + kg * 4;
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(W2 + (size_t)min(k + j, f - 1) * d);
                w2[q][j] = k < f ? v : zero;
            }
        if (bias1) bv = *reinterpret_cast<const f32x2_t*>(bias1 + (size_t)g * f + nc);
        zero_dropped();
        f32x4_t h[4][MS][2];                                     // every 16 k on their own: as few steps that round a sum as in the split products
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int ms = 0; ms < MS; ++ms) h[q][ms][0] = h[q][ms][1] = zero;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int ms = 0; ms < MS; ++ms) h[q][ms][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q][ms][j], w1[q][j][i], h[q][ms][i], 0, 0, 0);
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int i = 0; i < 2; ++i) h[0][ms][i] = (h[0][ms][i] + h[1][ms][i]) + (h[2][ms][i] + h[3][ms][i]);
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int r = 0; r < 4; ++r) {                        // D: rows 4 kg + r, column c
                const f32x2_t v = {gelu_tanh(h[0][ms][0][r] + bv[0]), gelu_tanh(h[0][ms][1][r] + bv[1])};
                *reinterpret_cast<f32x2_t*>(hs + (ms * 16 + kg * 4 + r) * HS + c * 2) = n < f ? v : f32x2_t{0.f, 0.f};
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();                         // another lane's values, the same wave's LDS operations: in order
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            f32x4_t hv[MS];
#pragma unroll
            for (int ms = 0; ms < MS; ++ms) hv[ms] = *reinterpret_cast<const f32x4_t*>(hs + (ms * 16 + c) * HS + q * 16 + kg * 4);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int ms = 0; ms < MS; ++ms) acc[q][ms][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(hv[ms][j], w2[q][j][i], acc[q][ms][i], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();                         // the piece is read before the sums are written over it
    } else {
        zero_dropped();
    }
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[0][ms][i] += acc[1][ms][i];
#pragma unroll
        for (int r = 0; r < 4; ++r) part[w][ms * 16 + kg * 4 + r][c] = f32x4_t{acc[0][ms][0][r], acc[0][ms][1][r], acc[0][ms][2][r], acc[0][ms][3][r]};
    }
    __syncthreads();
    const int row = tid / 16, n = (tid & 15) * 4;
    if (m0 + row >= rows || row >= MS * 16 || n >= d) return;
    f32x4_t v = part[0][row][tid & 15];
#pragma unroll
    for (int s = 1; s < kFWaves; ++s) v += part[s][row][tid & 15];
    f32_finish<EPI>(b, g, m0 + row, n, v);
}

template <int EPI> int launch_ffn_epi(const GemmArgs& a, const GemmArgs& b, hipStream_t s) {
    // A full 32-row tile keeps its compute unit's matrix cores busy for 4 us; 16-row ones as long as there are units for them
    // (256 tokens, 64/256, 8 experts x 32 rows 10.2 -> 8.3 us; 1500 tokens, top-2 of 16, dense branch 10.8 + 10.8 -> 8.0 + 8.0)
    const int tm = a.max_rows <= 16 || (long long)a.G * ((a.max_rows + 15) / 16) <= 256 ? 16 : 32;
    const long long tiles = ((long long)a.max_rows + tm - 1) / tm;
    if (tiles * 512 > 0xffffffffll) return MOE_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)tiles, (unsigned)a.G), block(kFWaves * 64);
    if (tm == 16) hipLaunchKernelGGL((f32_ffn_kernel<1, EPI>), grid, block, 0, s, a, b);
    else hipLaunchKernelGGL((f32_ffn_kernel<2, EPI>), grid, block, 0, s, a, b);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

template <int W, int EPI> int launch_rows_split(const GemmArgs& a, const dim3& grid, int n_tiles, hipStream_t s) {
    static OncePerDevice asked;
    const int rc = ask_lds(reinterpret_cast<const void*>(&f32_rows_split_kernel<W, EPI>), rows_split_lds<W>(), asked);
    if (rc != MOE_OK) return rc;
    hipLaunchKernelGGL((f32_rows_split_kernel<W, EPI>), grid, dim3(W * 64), rows_split_lds<W>(), s, a, n_tiles);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// The kernel of a product and its tile.
struct F32Choice {
    F32Kernel kernel;
    int rows, cols;
};
F32Choice pick_f32(const GemmArgs& a) {
    // Few tiles leave compute units idle, and the 32 x 64 ones of the rows kernels are four times as many.  They cost more per
    // flop, so the line is where two of them on every unit hold all (products, us, 32 x 64 / 64 x 128, both split: 2048 x 512, 256
    // small tiles 22 / 38, 512 tiles 38 / 38, with half of them empty 34 / 37; 512 x 2048, 384 tiles 12.4 / 15.0).
    const long long small_tiles = ((long long)a.max_rows + 31) / 32 * (((long long)a.N + 63) / 64) * a.G;
    const int expect = a.expect_rows > 0 && a.expect_rows < a.max_rows ? a.expect_rows : a.max_rows;
    // tiles if the rows fall evenly on the groups
    auto live = [&](int rows, int cols) { return (long long)a.G * ((expect + rows - 1) / rows) * (((long long)a.N + cols - 1) / cols); };
    if (a.max_rows <= 32 || small_tiles <= 512 || a.N >= 1 << 24) {
        if (a.max_rows <= 16) return {F32_ROWS16, 16, 64};
        if (a.K < 512 || a.N >= 1 << 24) return {F32_ROWS32, 32, 64};
        return {live(32, 64) > 256 ? F32_ROWS_SPLIT4 : F32_ROWS_SPLIT8, 32, 64};
    }
    // Split pieces or fp32 products, two small or one large work-group per compute unit (products, us, fp32 / split with two sets of waves /
    // with one): the split kernel's set-up and epilogue want a long K (4 x 2000, 200 x 800 45.6 / 44.7 / 37.8; 31 x 265, 128 x 512 25.2 / 24.8 /
    // 22.7; 8 x 2000, 100 x 200 20.0 / 18.2 / 17.1; 8 x 300, 192 x 256, 80 tiles 12.6 / 11.2 / 12.8: the line was drawn with waves of 64 columns,
    // which were the slower ones below it, and below 160 one large column among values of one sign is 1.1 times as far off 64 bits) and more than half a tile of columns (8 x 8192, 256 x 64 29 / 49 / 38).  One set leaves
    // room for a second work-group, whose products run under the first one's set-up and epilogue, but two of few tiles may meet on a
    // unit while another has none (8 x 384, 512 x 2048, 768 tiles 64 / 53 / 48; 4 x 480 with room for 720, 2048 x 1024, 256 tiles 75 / 53 / 80;
    // 31 x 132, 2048 x 512, 372 tiles 135 / 93 / 91).
    if (a.N <= 64) return {F32_TILE_NARROW, 128, 64};            // one 64-column tile: all four pairs of waves along the rows
    static_assert(kSRows == 64 && kSCols == 128, "the same tile");
    if (live(64, 128) > 256) return {a.K < 160 ? F32_TILE : F32_SPLIT1, 64, 128};
    return {a.K < 256 ? F32_TILE : F32_SPLIT2, 64, 128};
}

template <int EPI> int launch_epi(const GemmArgs& a, hipStream_t s) {
    const F32Choice c = pick_f32(a);
    const int n_tiles = (int)(((long long)a.N + c.cols - 1) / c.cols);
    const long long tiles = ((long long)a.max_rows + c.rows - 1) / c.rows * n_tiles;
    if (tiles * 512 > 0xffffffffll) return MOE_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)tiles, (unsigned)a.G), block(512);     // groups along y: x alone is limited to 2^32 threads, which E * capacity reaches
    static_assert(kFWaves * 64 == 512, "all unsplit kernels have the same work-group");
    switch (c.kernel) {
        case F32_ROWS16: hipLaunchKernelGGL((f32_rows_kernel<1, EPI>), grid, block, 0, s, a, n_tiles); break;
        case F32_ROWS32: hipLaunchKernelGGL((f32_rows_kernel<2, EPI>), grid, block, 0, s, a, n_tiles); break;
        case F32_ROWS_SPLIT8: return launch_rows_split<8, EPI>(a, grid, n_tiles, s);
        case F32_ROWS_SPLIT4: return launch_rows_split<4, EPI>(a, grid, n_tiles, s);
        case F32_TILE_NARROW: hipLaunchKernelGGL((f32_tile_kernel<4, 1, EPI>), grid, block, 0, s, a, n_tiles); break;
        case F32_TILE: hipLaunchKernelGGL((f32_tile_kernel<2, 2, EPI>), grid, block, 0, s, a, n_tiles); break;
        case F32_SPLIT1: return launch_split<1, EPI>(a, grid, n_tiles, s);
        case F32_SPLIT2: return launch_split<2, EPI>(a, grid, n_tiles, s);
        default: return MOE_ERR_INVALID_ARG;
    }
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

}  // namespace

// d_model up to 64 in one launch, against the two products (layers, us): d_ffn = 256, 8 experts, 256 tokens 24.3 / 21.1, 2048 27.9 /
// 24.2, 20000 52.5 / 46.1; 31 experts, top-2, 2048 tokens 38.5 / 31.8; 20/64 beside a dense branch, 1000 tokens 36.5 / 28.2.  Beyond
// 1024 row tiles the products on their own are as fast (65536 tokens 96.1 / 97.2), and with a longer d_ffn one work-group's rounds
// are the longer chain (256 tokens, 512: 25.0 / 26.0, 1024: 30.2 / 36.1).
bool ffn_f32_fused(const GemmArgs& a) { return a.K <= 64 && a.N <= kFWaves * 32 && (long long)a.G * ((a.max_rows + 31) / 32) <= 1024; }
int launch_ffn_f32(const GemmArgs& a, const GemmArgs& b, int epi, hipStream_t s) {
    if (a.max_rows <= 0 || a.G <= 0) return MOE_OK;
    if (a.K % 4 || a.N % 4 || !ffn_f32_fused(a) || b.K != a.N || b.N != a.K) return MOE_ERR_INVALID_ARG;
    switch (epi) {
        case EPI_STORE: return launch_ffn_epi<EPI_STORE>(a, b, s);
        case EPI_SCATTER: return launch_ffn_epi<EPI_SCATTER>(a, b, s);
        case EPI_COMBINE: return launch_ffn_epi<EPI_COMBINE>(a, b, s);
        default: return MOE_ERR_INVALID_ARG;
    }
}

F32Kernel f32_kernel(const GemmArgs& a) { return pick_f32(a).kernel; }

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
