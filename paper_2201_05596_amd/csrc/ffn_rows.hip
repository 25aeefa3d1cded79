// bf16 grouped GEMM for products that read few weights: a decode step with a handful of tokens, the dense branch of a
// decode step, the projections of a decoder block.  Bound by the read of the weights, and at these sizes by how many
// compute units share it: the streaming kernel (one wave per 128 columns over all of K) leaves a 1024 x 4096 product
// to 32 waves on one XCD.  Here a work-group of eight waves owns 16 NF columns and its waves split K between them:
//   * pairs of 32-deep k-blocks go to the waves in turn (a pair of blocks is a whole 128-byte line of every
//     activation row); weights and activations come straight from memory into registers, kAhead blocks ahead, and a wave's
//     last kAhead blocks fetch nothing (re-reading the last block kept the loop uniform and was a third to a half of the
//     loads of a short K: layers, us, 4 tokens, 1024/4096 beside a dense branch 37.9 -> 34.2, 64 tokens 142 -> 135; 64 tokens,
//     2048/8192, 128 experts 517 -> 510; with eight blocks ahead instead of four they are 3 to 10 % slower);
//   * the eight partial tiles are summed through LDS in wave order, so nothing depends on timing, and no partial
//     result passes through memory;
//   * consecutive work-groups (one per XCD) take different columns: one expert's weights are read by the whole chip;
//   * everything the epilogue needs from memory (bias, tokens and gate weights of the rows) is fetched first.
// Figures for the choice between this kernel, the streaming and the tiled one stand at rows_pick_* below.
#include <type_traits>

#include "ffn_common.h"

namespace moe {

namespace {

constexpr int kRWaves = 8;              // waves of a work-group = ways K is split
constexpr int kAhead = 4;               // k-blocks in flight per wave (even: a lane's pair of blocks stays together)

// NF 16-column fragments per work-group, at most 16 MSMAX rows per tile
template <int MSMAX, int NF, int EPI, bool PACKED>
__global__ __launch_bounds__(kRWaves * 64) void rows_kernel(const WsGemmArgs a0, const WsGemmArgs a1, const int split,
                                                            const int n_tiles, const int m_tiles0, const int m_tiles1) {
    constexpr int SUBS = MSMAX > 1 ? 2 : 1;                      // 16-row sub-tiles that one pass of the reduction finishes
    constexpr int COLS = 16 * NF;
    __shared__ __attribute__((aligned(16))) float part[kRWaves][SUBS * 16][COLS];

    const bool second = (int)blockIdx.x >= split;                // two products may share a launch (same K, N, packing)
    const WsGemmArgs& a = second ? a1 : a0;
    const int block = second ? (int)blockIdx.x - split : (int)blockIdx.x, m_tiles = second ? m_tiles1 : m_tiles0;
    const int tid = threadIdx.x, lane = tid & 63, c = lane & 15, kg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = block % n_tiles, mt = block / n_tiles % m_tiles, slot = block / n_tiles / m_tiles;
    const int g = a.order ? a.order[slot] : slot;
    const int rows = a.rows ? min(a.rows[g], a.max_rows) : a.fixed_rows;
    const int m0 = mt * MSMAX * 16, nrows = min(MSMAX * 16, rows - m0);

    // tokens that no expert kept have no other writer (top-1 combine): the work-group's first one is looked up here
    bool zero_first = false;
    if (EPI == EPI_SCATTER && a.zero_slot_idx) zero_first = (int)blockIdx.x < a.T && a.zero_slot_idx[blockIdx.x] < 0;

    auto run = [&](auto ms_count) {
        constexpr int MS = decltype(ms_count)::value;
        constexpr int PASSES = (MS + SUBS - 1) / SUBS;
        // this thread's part of the epilogue: row (tid / 16) of every pass, NF columns
        const int fr = tid >> 4, fc = tid & 15;
        const int n_fin = PACKED ? nt * NF / 8 * 128 + nt * NF % 8 + fc * 8 : nt * COLS + fc * NF;
        const bool fin = fr < SUBS * 16 && n_fin < a.N;
        int tok[PASSES];
        float gw[PASSES];
        float bias[NF];
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            tok[p] = 0;
            gw[p] = 1.f;
            if (EPI == EPI_SCATTER) scatter_lookup(a, g, m0 + min(p * SUBS * 16 + fr, nrows - 1), tok[p], gw[p]);
        }
        load_bias<NF>(a, g, min(n_fin, a.N - NF), bias);

        const uint16_t* a_src[MS];
#pragma unroll
        for (int ms = 0; ms < MS; ++ms) {                        // rows past the end repeat the last one
            const int r = m0 + min(ms * 16 + c, nrows - 1);
            const long long ar = a.row_map ? (long long)a.row_map[(size_t)g * a.map_stride + r] : (long long)g * a.a_group_stride + r;
            a_src[ms] = a.A + (size_t)ar * a.K + kg * 8;
        }
        const int nkb = (a.K + 31) / 32, p_ng = (a.N + 127) / 128;
        const uint16_t* B = PACKED ? a.B + (((size_t)g * nkb * p_ng + nt * NF / 8) * 8 + nt * NF % 8) * 512 + lane * 8
                                   : a.B + (size_t)g * a.K * a.N + min(nt * COLS + c * NF, a.N - NF);
        typedef typename std::conditional<NF == 8, uint4, typename std::conditional<NF == 4, uint2, uint32_t>::type>::type BRaw;
        struct Block {
            bf16x8_t av[MS], bf[PACKED ? NF : 1];
            BRaw braw[PACKED ? 1 : 8];
        };
        // wave w: blocks 2w, 2w + 1, 2w + 16, ...; past the end: in bounds (clamped), never multiplied
        const int whole = nkb / (2 * kRWaves), rest = nkb - whole * 2 * kRWaves;
        const int mine = __builtin_amdgcn_readfirstlane(whole * 2 + max(0, min(2, rest - 2 * w)));
        auto load = [&](Block& b, int i) {
            const int kb = min((i >> 1) * (2 * kRWaves) + w * 2 + (i & 1), nkb - 1);
            const int k = kb * 32 + kg * 8;                      // K is a multiple of 8: a lane's k are all inside or all outside
            const bool in = k < a.K;
#pragma unroll
            for (int ms = 0; ms < MS; ++ms)
                b.av[ms] = *reinterpret_cast<const bf16x8_t*>(a_src[ms] + (in ? kb * 32 : a.K - 8 - kg * 8));
            if constexpr (PACKED) {
                const uint16_t* p = B + (size_t)kb * p_ng * 4096;
#pragma unroll
                for (int j = 0; j < NF; ++j) b.bf[j] = __builtin_bit_cast(bf16x8_t, load_stream16(p + j * 512));
            } else {
                const uint16_t* p = B + (size_t)min(k, a.K - 8) * a.N;
#pragma unroll
                for (int j = 0; j < 8; ++j) b.braw[j] = *reinterpret_cast<const BRaw*>(p + (size_t)j * a.N);
            }
        };
        f32x4_t acc[MS][NF];
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int i = 0; i < NF; ++i) acc[ms][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        auto multiply = [&](Block& b, int i) {
            const int kb = (i >> 1) * (2 * kRWaves) + w * 2 + (i & 1);
            const bool in = kb * 32 + kg * 8 < a.K;              // false only in the last block of a ragged K
#pragma unroll
            for (int ms = 0; ms < MS; ++ms)
                if (!in) b.av[ms] = __builtin_bit_cast(bf16x8_t, make_uint4(0, 0, 0, 0));
            if constexpr (!PACKED) {                             // zeros on both sides: 0 times infinity is NaN
                if (kb * 32 + 32 > a.K) {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (!in) b.braw[j] = BRaw{};
                }
            }
            if constexpr (PACKED) {                              // zeros past K by themselves
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int ms = 0; ms < MS; ++ms)
                        acc[ms][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.av[ms], b.bf[f], acc[ms][f], 0, 0, 0);
            } else {
#pragma unroll
                for (int qq = 0; qq < NF / 2; ++qq) {            // 8 k-rows x 2 columns -> two fragments
                    uint32_t lo[4], hi[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const uint32_t r0 = raw_dword(b.braw[2 * p], qq), r1 = raw_dword(b.braw[2 * p + 1], qq);
                        lo[p] = __builtin_amdgcn_perm(r1, r0, 0x05040100u);
                        hi[p] = __builtin_amdgcn_perm(r1, r0, 0x07060302u);
                    }
                    const bf16x8_t blo = __builtin_bit_cast(bf16x8_t, make_uint4(lo[0], lo[1], lo[2], lo[3]));
                    const bf16x8_t bhi = __builtin_bit_cast(bf16x8_t, make_uint4(hi[0], hi[1], hi[2], hi[3]));
#pragma unroll
                    for (int ms = 0; ms < MS; ++ms) {
                        acc[ms][2 * qq] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.av[ms], blo, acc[ms][2 * qq], 0, 0, 0);
                        acc[ms][2 * qq + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.av[ms], bhi, acc[ms][2 * qq + 1], 0, 0, 0);
                    }
                }
            }
        };

        Block st[kAhead];
#pragma unroll
        for (int s = 0; s < kAhead; ++s) load(st[s], s);
        int i = 0;
        for (; i + kAhead < mine; i += kAhead) {             // the last round fetches nothing
#pragma unroll
            for (int s = 0; s < kAhead; ++s) {
                multiply(st[s], i + s);
                __builtin_amdgcn_sched_barrier(0);
                load(st[s], i + s + kAhead);
                __builtin_amdgcn_sched_barrier(0);               // the refill stays here, kAhead blocks before its use
            }
        }
#pragma unroll
        for (int s = 0; s < kAhead; ++s)
            if (i + s < mine) multiply(st[s], i + s);

#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            if (p > 0) lds_barrier();                            // the previous pass has been read
#pragma unroll
            for (int u = 0; u < SUBS; ++u) {
                if (p * SUBS + u >= MS) break;
#pragma unroll
                for (int r = 0; r < 4; ++r)                      // D: rows 4 (lane / 16) + r, column lane % 16
#pragma unroll
                    for (int f = 0; f < NF; ++f) part[w][u * 16 + kg * 4 + r][c * NF + f] = acc[p * SUBS + u][f][r];
            }
            lds_barrier();
            const int rl = p * SUBS * 16 + fr;
            if (fin && rl < nrows && rl < MS * 16) {
                float v[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) v[f] = 0.f;
#pragma unroll
                for (int s = 0; s < kRWaves; ++s)
#pragma unroll
                    for (int f = 0; f < NF; ++f) v[f] += part[s][fr][fc * NF + f];
#pragma unroll
                for (int f = 0; f < NF; ++f) v[f] += bias[f];
                if (EPI == EPI_STORE && a.partial) {             // the dense branch's sums, unrounded, for the combine
                    float* o = a.partial + (size_t)(m0 + rl) * a.N + n_fin;
#pragma unroll
                    for (int f = 0; f < NF; ++f) o[f] = v[f];
                } else {
                    finish_row<EPI, NF, true>(a, g, m0 + rl, 0, n_fin, v, tok[p], gw[p]);
                }
            }
        }
    };
    if (nrows > 0) {
        if (MSMAX == 1 || nrows <= 16) run(std::integral_constant<int, 1>());
        else if (MSMAX == 2 || nrows <= 32) run(std::integral_constant<int, MSMAX < 2 ? MSMAX : 2>());
        else run(std::integral_constant<int, MSMAX>());
    }
    if (EPI == EPI_SCATTER && a.zero_slot_idx) {
        for (int t = blockIdx.x; t < a.T; t += gridDim.x) {
            if (t != (int)blockIdx.x ? a.zero_slot_idx[t] < 0 : zero_first) {
                uint4* o = reinterpret_cast<uint4*>(a.out + (size_t)t * a.N);
                for (int i = tid; i < a.N / 8; i += kRWaves * 64)
                    o[i] = a.add ? reinterpret_cast<const uint4*>(a.add + (size_t)t * a.N)[i] : make_uint4(0, 0, 0, 0);
            }
        }
    }
}

inline int rows_slots(const WsGemmArgs& a) { return a.order && a.slots > 0 && a.slots < a.G ? a.slots : a.G; }

template <int MSMAX, int NF, int EPI, bool PACKED>
int launch_r(const WsGemmArgs& a, const WsGemmArgs* b, hipStream_t s) {
    const int n_tiles = PACKED ? (a.N + 127) / 128 * (8 / NF) : (a.N + 16 * NF - 1) / (16 * NF);
    const int m0 = (a.max_rows + MSMAX * 16 - 1) / (MSMAX * 16), m1 = b ? (b->max_rows + MSMAX * 16 - 1) / (MSMAX * 16) : 1;
    const long long blocks_a = (long long)rows_slots(a) * m0 * n_tiles, blocks_b = b ? (long long)rows_slots(*b) * m1 * n_tiles : 0;
    if (blocks_a + blocks_b > (1ll << 30)) return MOE_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((rows_kernel<MSMAX, NF, EPI, PACKED>), dim3((unsigned)(blocks_a + blocks_b)), dim3(kRWaves * 64), 0, s, a,
                       b ? *b : a, (int)blocks_a, n_tiles, m0, m1);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

template <int NF, int EPI, bool PACKED>
int launch_r_rows(const WsGemmArgs& a, const WsGemmArgs* b, hipStream_t s) {
    const int most = b && b->max_rows > a.max_rows ? b->max_rows : a.max_rows;
    if (most <= 16) return launch_r<1, NF, EPI, PACKED>(a, b, s);
    if (most <= 32) return launch_r<2, NF, EPI, PACKED>(a, b, s);
    return launch_r<4, NF, EPI, PACKED>(a, b, s);
}

template <int EPI>
int launch_r_epi(const WsGemmArgs& a, const WsGemmArgs* b, int NF, hipStream_t s) {
    if (!a.packed) return NF == 2 ? launch_r_rows<2, EPI, false>(a, b, s) : launch_r_rows<4, EPI, false>(a, b, s);
    if (NF == 1) return launch_r_rows<1, EPI, true>(a, b, s);
    if (NF == 2) return launch_r_rows<2, EPI, true>(a, b, s);
    return launch_r_rows<4, EPI, true>(a, b, s);
}

}  // namespace

// ---- where this kernel is the faster one, and with how many columns per work-group -----------------------------------
// All figures: us per layer call on packed weights unless said otherwise, this kernel against the one it stands in for.

// Columns: the most that leave 160 work-groups (64 of 16 columns where there are no more); 64 columns read whole 4 KB
// pieces of packed weights, fewer put more compute units on the same bytes.  Dense branch, d = 2048, 64 rows, GEMM-1
// with 16 / 32 / 64 columns: 502 / 491 / 495; 128 rows: 506 / 484 / 486; GEMM-2, 64 rows: 415 / 420 / 430, 256 rows:
// 487 / 453 / 461.
static int rows_columns(long long groups, int max_rows, int N, bool packed) {
    const long long m_tiles = max_rows <= 32 ? 1 : (max_rows + 63) / 64;
    for (int nf = 4; nf > 1; nf /= 2)
        if (groups * m_tiles * ((N + 16 * nf - 1) / (16 * nf)) >= 160) return nf;
    return packed ? 1 : 2;
}

// Experts' first product, against the streaming kernel.  That one has a wave per 128 columns: with slots x N up to 48 K
// columns it leaves compute units idle (1 token, 1024 x 4096: 22.8 -> 5 us in this kernel; 2048 x 8192, 2 tokens 87 -> 39
// with both products; plain weights 12 tokens of d = 1024: 67.1 / 67.0, 16: 70.8 / 75.8).  Beyond, with packed weights and K >=
// 2048, what decides is how many experts the tokens reach: the streaming kernel deals whole experts to the eight XCDs, so a
// number that is no multiple of eight leaves some XCDs idle at the end.  While the tokens are few enough to miss experts
// (up to two choices per expert) this kernel wins (2048 x 8192: 64 tokens, 32 experts 158 / 150; 64, 64: 204 / 194; 16, 16:
// 65 / 53; 64 tokens, 128 experts, of which about 51 are reached: layer 519 / 506; where they happen to be 48: 242 / 246 for the
// product); with all of a multiple of eight experts reached, or fewer than eight of them, the streaming one does (128 tokens,
// 8 experts 44 / 52; 64, 16: 86 / 88).  with_dense: the dense branch's first product comes along in the launch, which pays for it
// (block of 10 tokens, top-2 of 8 experts, 2048 / 8192: 122 / 138).
//
// K below 2048, where a work-group's waves have four blocks each, and up to 256 rows: as long as few experts have more than one (layers,
// even routing and with gate bias 1.5 ln(1 / (e + 1)), streaming / this kernel: 16 tokens, 1024 / 4096, 64 experts 57.6 / 53.4 and
// 38.8 / 22.7; 64 tokens, 128 experts 141 / 139 and 42.6 / 28.5; 180 tokens, 128 experts -4 % and -10 %; 64 tokens of 32 87.9 / 89.0, 34.2 /
// 24.6; 20 tokens, top-2 of 32 +2 % and -19 %).
int rows_pick_gemm1(long long touched, int max_rows, long long kept, int K, int N, bool packed, bool with_dense) {
    if (max_rows > 16) return 0;
    if (touched * N > 48 * 1024) {
        if (!packed) return 0;
        const bool spread = 2 * kept < 3 * touched;                // few experts have more than one row
        if (K < 1024 || kept > (spread ? 256 : 128)) return 0;
        if (K < 2048 && (kept >= 2 * touched || (touched < 64 && 4 * kept >= 5 * touched))) return 0;
        if (K >= 2048 && !with_dense && kept > 2 * touched && (touched % 8 == 0 || touched < 8)) return 0;
    }
    const int nf = rows_columns(touched, max_rows, N, packed);
    return packed ? nf : 4;                                    // plain rows of 64 bytes: 4 tokens, d = 2048, 110 against 91
}

// Experts' second product, against the streaming kernel with K split over work-groups and a kernel that adds up
// (few_waves): 64 tokens, 128 experts, d = 1024 166 -> 156, 96 tokens, 64 experts 158 -> 151; 48 tokens, d = 2048 464 ->
// 445; 256 tokens, 32 experts, top-2 (up to 32 rows each), d = 2048 382 -> 373.  With K < 8192 it is within 1 % either
// way from 128 rows on (120.2 / 119.0, 122.6 / 121.2, 216 / 218) and, where the streaming kernel needs no split, within
// 3 %: that one stays there.  With K < 8192 16 columns are the best split (32 experts, 32 rows, d = 1024: 75.2 / 79.3 /
// 83.9 with 16 / 32 / 64), many short work-groups of which four share a compute unit; longer ones want more (d = 2048:
// 245 / 242 / 251; 256 rows of 32 experts, top-2: 457 / 395 / 373; K = 16384, 8 experts, 128 tokens 226 / 205 / 170; 12
// tokens, layer with 32 / 64 columns 225 / 241).  Every work-group reads the rows of its expert again, so many rows per
// expert, few columns per work-group and a long K lose to the streaming kernel's one pass: product with K = 8192, N =
// 2048, 1 expert of 64 rows 45 / 32, 4 of 64 54 / 41, of 32 38 / 36; K = 16384, N = 4096, 2 experts of 24 rows 62 / 54,
// 1 of 64 82 / 50; K = 4096, N = 1024, 1 of 64 26.5 / 22.5.
// Plain weights (rows of 64 bytes, so twice the lines are touched): one or two experts only, and with a long K only out of at
// least eight (fewer are spread over the XCDs by columns: K = 8192, 2 experts of 16 rows 31 / 27, K = 16384, 1 of 16 54 / 40; 2
// tokens out of 8 experts, 2048 / 8192: layer 44 / 59).
// At most 16 rows per expert, packed, against the streaming kernel without a split as well: that one's waves are then enough for the
// chip only if all experts have rows, and with skewed routing most have none.  With few rows per expert (whatever few_waves says) or, K
// below 8192, up to 256 rows (layers, us, even routing and with gate bias 1.5 ln(1 / (e + 1)), streaming / this kernel: 2048 / 8192, 64
// tokens of 64 experts 453 / 423 and 136 / 70, 96 of 128 729 / 664 and 203 / 85, 180 of 128 974 / 959 and 224 / 112, 40 tokens, top-2 of
// 64 484 / 484 and 156 / 106, but 90 of 64 522 / 525; 1024 / 4096, 180 of 128 280 / 261 and 88 / 44, 100 tokens, top-2 of 64 180 / 174 and 50 / 43; with 32 columns
// 180 of 128 962 / 980).  Not with fewer tokens than three quarters of the experts, where even routing loses what it gains elsewhere (64
// of 128 498 / 507, skewed 196 / 76), nor with two rows per expert and more (+1 .. +4 %, skewed -17 .. -38 %).
int rows_pick_gemm2(int E, long long touched, int max_rows, long long kept, int K, int N, bool packed, bool few_waves) {
    const bool few_rows = max_rows <= 16;
    const bool spread = touched >= 96 ? 2 * kept < 3 * touched : 4 * kept <= 5 * touched;      // few experts have more than one row
    if (packed && few_rows && !few_waves && kept <= 256 && spread && 4 * kept >= 3ll * E) return 1;
    if (!few_waves || kept > (K >= 8192 || (packed && few_rows) ? 256 : 96)) return 0;
    if (!packed) return (K < 8192 || E >= 8) && few_rows && touched * N <= 4096 ? 2 : 0;
    int nf = rows_columns(touched, max_rows, N, packed);
    if (few_rows) return K < 8192 ? 1 : nf > 2 && (K < 16384 || kept < 8 * touched) ? 2 : nf;
    if (K < 8192) return K >= 4096 && kept > 48 * touched ? 0 : nf;
    if (kept > 16 * touched && (max_rows > 32 || nf == 2)) return 0;
    return kept > 24 * touched && nf < 4 ? 0 : nf;
}

// Dense branch, against the streaming kernel (up to 64 tokens: one wave per 128 columns; GEMM-2 of 16 tokens, d = 2048:
// 98 -> 11 us) and the tiled one (up to 32 tiles of 128 x 256 would do the work, T x N up to 1 M): GEMM-2, d = 1024, 800
// tokens 455 -> 426, 1100: 466 -> 470; GEMM-1, d = 2048, 128 tokens 505 -> 485, 200: 507 -> 511.
int rows_pick_dense(int T, int N, bool packed) {
    return (long long)T * N <= 1 << 20 ? rows_columns(1, T, N, packed) : 0;
}

int launch_rows(const WsGemmArgs& a, const WsGemmArgs* b, int epi, int NF, hipStream_t s) {
    if (a.G <= 0 || a.max_rows <= 0) return MOE_OK;
    if (a.ksplit != 1 || !wsgemm_supported(a.K, a.N)) return MOE_ERR_INVALID_ARG;
    if (b && (epi == EPI_SCATTER || b->K != a.K || b->N != a.N || (b->packed != 0) != (a.packed != 0))) return MOE_ERR_INVALID_ARG;
    switch (epi) {
        case EPI_STORE: return launch_r_epi<EPI_STORE>(a, b, NF, s);
        case EPI_GELU: return launch_r_epi<EPI_GELU>(a, b, NF, s);
        case EPI_SCATTER: return launch_r_epi<EPI_SCATTER>(a, b, NF, s);
        case EPI_COMBINE: return launch_r_epi<EPI_COMBINE>(a, b, NF, s);
        default: return MOE_ERR_INVALID_ARG;
    }
}

}  // namespace moe
