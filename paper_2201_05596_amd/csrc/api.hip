// C ABI of the library: argument checks, workspace carving and launch sequencing.
// Every check happens on the host before the first HIP call.
#include <algorithm>
#include <vector>

#include "call_tag.h"
#include "moe_internal.h"

using namespace moe;

namespace {

// ---- optional stage timing of moe_layer_forward (benchmark aid) ----------------------------------
// When enabled, an event is recorded on the call's stream before the first kernel and after every
// stage; nothing is read back until moe_profile_elapsed() is called.
enum Stage { ST_LOGITS, ST_ROUTE, ST_DISPATCH, ST_GEMM1, ST_GEMM2, ST_REDUCE, ST_DENSE1, ST_DENSE2, ST_COMBINE, ST_COUNT };
const char* const kStageNames[ST_COUNT] = {"gate_logits", "gate_route", "dispatch", "expert_gemm1", "expert_gemm2",
                                           "splitk_reduce", "dense_gemm1", "dense_gemm2", "combine"};
struct Profiler {
    int max_calls = 0, calls = 0, cur = -1;
    int stride = 1, seen = 0;       // only every stride-th call since the last enable is timed
    unsigned mask = ~0u;            // stages that get their own time
    bool dirty = false;             // kernels were launched since the last recorded event
    std::vector<hipEvent_t> ev;     // [max_calls][kMarks]
    std::vector<int> stage;         // stage that ended at each mark; -1: the mark only opens the next stage
    std::vector<int> nmarks;        // [max_calls]
} g_prof;
constexpr int kMarks = 2 * ST_COUNT + 1;

void prof_record(int stage, hipStream_t st) {
    const int m = g_prof.nmarks[g_prof.cur];
    if (m >= kMarks) return;
    g_prof.stage[(size_t)g_prof.cur * kMarks + m] = stage;
    (void)hipEventRecord(g_prof.ev[(size_t)g_prof.cur * kMarks + m], st);
    g_prof.nmarks[g_prof.cur] = m + 1;
    g_prof.dirty = false;
}
void prof_begin(hipStream_t st) {
    g_prof.cur = -1;
    if (g_prof.max_calls == 0 || g_prof.calls >= g_prof.max_calls) return;
    if (g_prof.seen++ % g_prof.stride != 0) return;
    g_prof.cur = g_prof.calls++;
    g_prof.nmarks[g_prof.cur] = 0;
    g_prof.dirty = true;            // whatever ran before the call
}
// before a stage's first launch: open it with an event unless one was just recorded
void prof_pre(int stage, hipStream_t st) {
    if (g_prof.cur < 0 || !(g_prof.mask >> stage & 1u)) return;
    if (g_prof.dirty || g_prof.nmarks[g_prof.cur] == 0) prof_record(-1, st);
}
// after a stage's last launch
void prof_mark(int stage, hipStream_t st) {
    if (g_prof.cur < 0) return;
    if (g_prof.mask >> stage & 1u) prof_record(stage, st);
    else g_prof.dirty = true;
}

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t esize(int dtype) { return dtype == MOE_F32 ? 4 : 2; }

int check_shape(const moe_shape_t* s) {
    if (!s) return MOE_ERR_INVALID_ARG;
    if (s->T < 1 || s->d_model < 1 || s->d_ffn < 1 || s->E < 1 || s->capacity < 1) return MOE_ERR_INVALID_ARG;
    if (s->top_k < 1 || s->top_k > s->E) return MOE_ERR_INVALID_ARG;
    if (s->dtype != MOE_F32 && s->dtype != MOE_BF16) return MOE_ERR_INVALID_ARG;
    if (s->residual != 0 && s->residual != 1) return MOE_ERR_INVALID_ARG;
    if (s->flags & ~(MOE_FLAG_PACKED_WEIGHTS | MOE_FLAG_PACKED_GATE)) return MOE_ERR_INVALID_ARG;
    if ((s->flags & MOE_FLAG_PACKED_WEIGHTS) && s->dtype != MOE_BF16) return MOE_ERR_UNSUPPORTED;
    if ((s->flags & MOE_FLAG_PACKED_GATE) && (s->dtype != MOE_BF16 || !gate_bf16_supported(s->d_model, s->E)))
        return MOE_ERR_UNSUPPORTED;
    if (s->top_k > 2 || s->E > 1024) return MOE_ERR_UNSUPPORTED;
    const int mult = s->dtype == MOE_F32 ? 4 : 8;
    if (s->d_model % mult || s->d_ffn % mult) return MOE_ERR_UNSUPPORTED;
    if ((long long)s->T * s->top_k >= (1ll << 31) || (long long)s->E * s->capacity >= (1ll << 31))
        return MOE_ERR_UNSUPPORTED;
    return MOE_OK;
}

// Tile shapes and split-K factor of the two expert GEMMs (bf16 MFMA path).
struct FfnPlan {
    bool mfma;          // false: the fp32 kernels (fp32 layers)
    int MT, NW1, NW2;   // row tile; waves per work-group of GEMM-1 / GEMM-2
    int ksplit2;        // split-K factor of GEMM-2 (1 = none)
    int ksplit_room;    // split-K factor that the workspace has room for
    bool tiled;         // the tiled kernel: more than 64 rows per expert, or packed weights and enough tiles (few_rows_tiled)
    bool tiled1;        // the tiled kernel for GEMM-1, whatever GEMM-2 takes
    int NBUF;           // weight super-fragments kept in flight per wave, plus one
    int nf1, nf2;       // 16-column fragments per work-group of the few-weights kernel, 0: not that kernel
    int slots;          // launch-order entries that may have rows, 0: all
    int expect;         // rows per expert if the tokens fall evenly on them
};

// Experts with room for at most 64 rows: both kernels read the weights once, and on packed ones the tiled kernel does it
// faster (whole 32 KB blocks by direct loads, no sums of partial results) if there are tiles enough for the compute units: its
// tiles are as long as K, where the streaming kernel splits that.  How many have rows depends on the routing, which the host does
// not know: over 1005 layers (1024 to 4096 wide, 16 to 256 experts, 2 to 62 rows per expert) the products that these rules put on
// tiles take 0.97 of the streaming kernel's time with even routing, 0.90 with gate bias ln(1 / (e + 1)) and 0.83 with 1.5 of it, but
// 4 % of the layers lose more than 3 %, where the tiles of a few busy experts just miss a round: at most 1.20 (4096/4096, 100
// experts x 7 rows of which 17 hold 86, 204 / 245 us), one product 1.41 (2048 x 8192, 9 of 256 experts hold 35 rows, 63 / 90).
// Layers, us or per cent of the streaming kernel's time:
//   first product (d_ffn columns): from 3 rows per expert on, 8 of fewer than 32 experts.  64 experts x 22 .. 45 rows (1024/4096)
//     with skewed routing -12 .. -14 %, 32 x 24 -5 %, 2048/8192 64 x 58 -5 %, even routing -3 .. +0 %; 92 tokens of 64 experts
//     144 / 152;
//   both products: from 512 tiles in the second one on, with 7/4 rows per expert (so that few are missed).  128 x 33 rows
//     (1024/4096) skewed 135 / 104, even 382 / 374; 2048/8192 64 x 58 skewed 247 / 206, 64 x 24 even 668 / 643; 256 tokens of 128
//     experts 313 / 303, 164 tokens 250 / 252.  With half the tiles even routing gains (64 x 64, 1024/4096, 235 / 206) but a few
//     busy experts lose (64 x 45 85 / 94, 64 x 7 60 / 75, 40 x 55 72 / 93), and so does 4096/16384 (64 x 5 skewed 800 / 844).  Beside a
//     dense branch, whose products keep launches of their own: 1000 tokens of 64 experts, 2048/8192, 786 / 777, skewed 327 / 313;
//     3000 tokens, top-2 of 128, 1024/4096, 470 / 473, skewed 216 / 182; 151 tokens of 64 660 / 639, skewed 228 / 211.  With at most
//     128 tokens such layers stay on the streaming kernel, though tiles are not slower there (112 tokens of 64 572 / 569, skewed
//     221 / 209);
//   more than 48 rows on a short K leave the set-up and epilogue of a tile too little to hide behind: 128 x 64 (1024/4096)
//     394 / 404, 128 x 33 .. 38 -0.1 .. -2 %.
bool few_rows_short(const moe_shape_t* s) { return !(s->flags & MOE_FLAG_PACKED_WEIGHTS) || (s->capacity > 48 && s->d_model < 2048); }
bool few_rows_tiled(const moe_shape_t* s, long long kept) {
    if (few_rows_short(s) || (s->residual && s->T <= 128)) return false;
    return (long long)s->E * ((s->d_model + 255) / 256) >= 512 && s->d_ffn <= 8192 && 4 * kept >= 7ll * s->E;
}

FfnPlan plan_ffn(const moe_shape_t* s) {
    FfnPlan p{};
    p.mfma = s->dtype == MOE_BF16 && wsgemm_supported(s->d_model, s->d_ffn);
    p.ksplit2 = p.ksplit_room = 1;
    p.NBUF = 2;
    if (!p.mfma) return p;
    const long long kept = (long long)s->T * s->top_k, touched = s->E < kept ? s->E : kept;
    p.expect = (int)((kept + s->E - 1) / s->E < s->capacity ? (kept + s->E - 1) / s->E : s->capacity);
    const bool tiles_fit = tgemm_supported(s->d_model, s->d_ffn) && tgemm_supported(s->d_ffn, s->d_model);
    p.tiled = tiles_fit && (s->capacity > 64 || few_rows_tiled(s, kept));
    // Few experts, an inner dimension off the 32-deep stages and a long second product: on the tiled kernel that one leaves most
    // of the chip idle, the streaming kernel splits its K (1000 / 4000, plain, 2 experts x 156 rows: layer 92 us tiled, 78
    // streamed; 2008 / 8032, 1 x 128: 161 / 116; 72 / 2088, 8 x 160: 57 / 47).  The tiled one is the faster with more rows (1 x
    // 1000 of 1000: 97 / 120), from about 64 tiles of 128 x 128 on (4 x 400: 99 / 137; 64 experts x 65 of 72 / 2088: 60 / 72) and
    // where the second product is not much the longer one (4 x 128 of 1000 / 1000: 54 / 63).  Whole stages are not asked here:
    // they always went to the tiled kernel.
    const bool whole_stages = s->d_model % 32 == 0 && s->d_ffn % 32 == 0;
    const long long tiles2 = (long long)s->E * ((s->capacity + 127) / 128) * ((s->d_model + 127) / 128);
    if (!whole_stages && s->capacity <= 512 && s->E <= 32 && tiles2 <= 64 && s->d_ffn >= s->d_model + 2000) p.tiled = false;
    p.tiled1 = p.tiled || (tiles_fit && s->capacity <= 64 && s->E >= 16 && p.expect >= (s->E >= 32 ? 3 : 8) && !few_rows_short(s));
    wsgemm_pick_tile(s->capacity, s->E, s->d_ffn, &p.MT, &p.NW1);
    int mt2;
    wsgemm_pick_tile(s->capacity, s->E, s->d_model, &mt2, &p.NW2);
    // GEMM-2 has few output columns; when that leaves the chip short of waves, split K
    const long long m_tiles = (s->capacity + p.MT - 1) / p.MT;
    const long long waves = touched * ((s->d_model + 127) / 128) * m_tiles;
    const bool packed = s->flags & MOE_FLAG_PACKED_WEIGHTS;
    if (s->capacity <= 64) {
        p.nf1 = rows_pick_gemm1(touched, s->capacity, kept, s->d_model, s->d_ffn, packed, s->residual && s->T <= 16);
        p.nf2 = rows_pick_gemm2(s->E, touched, s->capacity, kept, s->d_ffn, s->d_model, packed, waves < 1024);
    }
    // The room for partial sums is that of the streaming kernel's split whether or not the call takes it, so that a
    // workspace sized for packed weights serves the same shape with plain ones (the few-weights kernel's rule knows them
    // apart) and no size depends on which kernel is the faster one.
    if (waves < 1024 && !(s->capacity > 64 && whole_stages)) {
        const int chunks = (s->d_ffn + wsgemm_chunk_k(p.MT) - 1) / wsgemm_chunk_k(p.MT);
        long long ks = (2048 + waves - 1) / waves;
        if (ks > 8) ks = 8;
        if (ks > chunks) ks = chunks;
        p.ksplit_room = (int)(ks < 1 ? 1 : ks);
        if (!p.tiled && !p.nf2) p.ksplit2 = p.ksplit_room;
    }
    return p;
}

// do the bf16 matrix cores compute the gate logits?
bool gate_on_bf16(const moe_shape_t* s) { return s->dtype == MOE_BF16 && gate_bf16_supported(s->d_model, s->E); }

// Does the dense branch's second product share the launch of the experts' in the few-weights kernel?  Both have to take that kernel:
// alone the dense one is a chain through all of K on few work-groups (16 tokens, 2048/8192 16 us, 96 tokens 42, for 34 MB of
// weights).  Its sums stay unrounded in 32 bits for the combine, which then is a launch of its own (4.7).  Layers, us, apart /
// shared: one token, 1024/4096, 64 experts 26.9 / 23.8; 16 tokens, 2048/8192, 64 experts 174.2 / 169.6, two tokens, plain weights
// 101.8 / 77.7; 40 tokens, 1024/4096, 128 experts 126 / 113; 96, top-2 of 32, skewed 196 / 169; 150 of 128 270 / 258.
// On packed weights and more than 1024 columns, where the dense one alone fills half the chip and more, not
//   - with fewer tokens than a 128th of the columns, unless all work-groups run at once: the dense ones make a round of their own, of the
//     experts' columns per work-group (apart / shared: 2048/8192, 2 tokens, top-2 of 32 71.4 / 78.0, one token, top-2 51.2 / 53.5, but top-1
//     44 / 41; 4096/16384, 2 of 16 142 / 154, 16 512 / 522, 32 the same; 1536/6144, one, top-2 of 32 1.08 times);
//   - with so many that reading their rows again in every work-group of few columns is what the launch takes (2048/4096, 256
//     tokens of 32, 16 columns 232 / 251, skewed 110 / 127; 2048/8192, 160 of 128, skewed 150 / 180, with 32 columns, 128 of 32 the same;
//     4096/8192, 96 of 16, 32 columns 1.03, 64 0.98 times);
//   - with a K below 4096 (2048/2048 1.00 to 1.12 times at 1 to 24 and 80 to 256 tokens).
// With up to 1024 columns it gains (0.78 to 1.00 times, 512/2048, 1000/4000, 1024/4096 .. 16384), but with many tokens and a shorter K (1024/4096,
// 256 of 32 137.8 / 140.1; 1024/256, 200 of 32 46.6 / 48.9).  Plain weights, which take that kernel for a few rows only: 0.68 to 1.00
// times but with many columns and a short K (2048/1024, one token, top-2 of 32 31.6 / 32.7, 4096/1024 37.5 / 40.7, 4096/4096 66.1 / 64.6).
constexpr int kSharedTokens = 256;             // the few-weights kernel takes no second products of more rows
bool dense2_shared(const moe_shape_t* s, const FfnPlan& p) {
    const bool packed = s->flags & MOE_FLAG_PACKED_WEIGHTS;
    if (!s->residual || s->T > kSharedTokens || !p.mfma || !p.nf2 || p.ksplit2 != 1 || !rows_pick_dense(s->T, s->d_model, packed)) return false;
    const long long T = s->T, N = s->d_model, K = s->d_ffn;
    if (!packed) return N <= 1536 || K >= N;
    if (N <= 1024) return K >= 8192 || T * N <= (K < 2048 ? 128 : 208) * 1024;
    const long long kept = T * s->top_k, touched = s->E < kept ? s->E : kept;
    const bool one_round = (touched + 1) * ((N + 16 * p.nf2 - 1) / (16 * p.nf2)) <= 256;
    const bool few_rows = N <= 2048 ? T * K <= p.nf2 << 19 : T <= 32 * p.nf2;
    return K >= 4096 && few_rows && (128 * T >= N || one_round);
}

// Where it does not: K split on the streaming kernel, whose sums the combine adds up (1: not that way).  For 33 to 192 tokens and a long K,
// where the few-weights kernel would take the product, every work-group of it reading 64 rows through all of K: layers, us, that
// kernel with the combine in it / split: 120 tokens, 2048/8192, top-2 of 64, skewed 225 / 215, 140 of 64, skewed 204 / 190;
// 180 tokens, 1024/4096, top-2 of 64 226 / 219; plain weights, 50 tokens, 2048/8192, top-2 of 32 401 / 392; but 256 tokens, 1024/4096,
// 137.8 / 138.7.  On packed weights from 41 tokens on: 33, 2048/8192, top-2 of 2 114.9 / 118.7, 36 118.6 / 120.3, 40 and 41 the
// same, 44 123.8 / 121.3, 4096/16384, 41 of 2 207.6 / 203.1; plain, 33 tokens, 2048/8192, top-2 of 8 150.7 / 149.2, 64 experts
// 349.3 / 346.9, 4096/16384, top-2 of 2 251.9 / 231.7, 1024/4096, top-2 of 32 122.8 / 122.2.
constexpr int kSplitTokens = 192;
int dense2_split(const moe_shape_t* s) {
    const bool packed = s->flags & MOE_FLAG_PACKED_WEIGHTS;
    if (s->T <= (packed ? 40 : 32) || s->T > kSplitTokens || s->d_ffn < 4096 || !rows_pick_dense(s->T, s->d_model, packed)) return 1;
    int MT, NW;
    wsgemm_pick_tile(s->T, 1, s->d_model, &MT, &NW);
    const long long waves = (long long)((s->d_model + 127) / 128) * ((s->T + MT - 1) / MT);
    const int chunks = (s->d_ffn + wsgemm_chunk_k(MT) - 1) / wsgemm_chunk_k(MT);
    const long long ks = (2048 + waves - 1) / waves < kLinearMaxSplit ? (2048 + waves - 1) / waves : kLinearMaxSplit;
    return (int)(ks > chunks ? chunks : ks);
}

// The waves' tiles of an expert GEMM-2 whose K is split on the streaming kernel: about 200 of its work-groups of two waves, the fewest
// of the numbers measured that lost nowhere.  The factor in the plan is for few experts with rows (2048 tiles, eight ways at most, of those that the
// tokens can reach at most); where all have some, it wrote and read more partial sums than the product gains.  Layers, us, the
// plan's factor / at least 600 tiles / at least 400, even routing: 1000/4000, plain, 40 experts x 64 rows 237 / 212 / 212; 32 x 20
// 123 / 121 / 112; 1024/4096, packed, 32 x 60 142 / 133 / 124; plain, 64 x 30 213 / 204 / 195; 4096/16384, 16 x 30 741 / 685 / 662; 16
// tokens of 64 experts 86 / 90 / 84.
// Experts of very different sizes (skewed routing) keep the plan's factor: with at least 400 423 tokens, 4096/16384, 16 experts beside a
// dense branch took 885 -> 899, with at least 300 100 tokens, 1000/4000, top-2 of 32 84 -> 87.  The host, which knows no routing,
// cannot choose: its own factor for 400 tiles took skewed 40 x 48 79 -> 87, 40 x 60 74 -> 93.
// Nor with few rows per expert, whose sums are few: below 3 on average (4096 columns and more: 3/2) the plan's factor is the faster one
// with even and slightly skewed routing.  Layers, us, the plan's factor / at least 400 tiles: 1024/4096, plain, 32 experts, 16
// tokens 55.9 / 58.0, 32 78.3 / 85.3, 48 89.6 / 91.6, but 96 102.6 / 100.4; 1000/4000, 30 of 40 96.3 / 107.2; 2048/8192, 8 of 16 96.1 / 103.1, 24
// 167.6 / 170.3, 48 189.0 / 179.0; 4096/16384, 2 of 16 173.9 / 182.4, 24 637 / 613.  And not where all experts together have too few tiles
// for another factor: looking for the count costs both kernels a round trip (512/2048, 32 experts, 192 tokens 42.5 / 43.4).
constexpr int kSplitTiles = 400;
int split_tiles(const moe_shape_t* s, const FfnPlan& p) {
    const long long kept = (long long)s->T * s->top_k, touched = s->E < kept ? s->E : kept;
    const long long waves = touched * ((s->d_model + 127) / 128);
    const bool one_row_tile = s->capacity <= p.MT, many_rows = s->d_model < 4096 ? kept >= 3ll * s->E : 2 * kept >= 3ll * s->E;
    return one_row_tile && many_rows && (kSplitTiles + waves - 1) / waves < p.ksplit2 ? kSplitTiles : 0;
}

// Carving of the caller's workspace.  Offsets in bytes; every region 256-byte aligned.
struct WsLayout {
    size_t logits, wg_frags, hist, flags, expert_idx, slot_idx, gate_w, rows, order, slot_token, h, ye, hd, dense, partial, total;
};

WsLayout ws_layout(const moe_shape_t* s) {
    WsLayout L{};
    const size_t T = s->T, d = s->d_model, f = s->d_ffn, E = s->E, k = s->top_k, C = s->capacity;
    const size_t es = esize(s->dtype);
    const FfnPlan plan = plan_ffn(s);
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += align_up(bytes); return o; };
    L.logits = take(T * E * 4);
    L.wg_frags = take(s->dtype == MOE_BF16 ? gate_bf16_ws_bytes(s->d_model, s->E) : 0);
    L.hist = take(route_scratch_ints(s->T, s->E, s->top_k, !gate_on_bf16(s)) * 4);
    // hand-over flags of the one-launch decode gate: it leaves no histograms, so they reach back into that region
    static_assert(kGateFlags * 8 <= 2 * kAlign, "at least one unit of histograms before the extra one");
    take(kAlign);
    L.flags = off - kGateFlags * 8;
    L.expert_idx = take(T * k * 4);
    L.slot_idx = take(T * k * 4);
    L.gate_w = take(T * k * 4);
    L.rows = take(E * 4);
    L.order = take(2 * (E + 1) * 4);  // two launch orders of the experts, each followed by the tile-dealing flag
    L.slot_token = take(E * C * 4);
    L.h = take(E * C * f * es);
    L.ye = take(E * C * d * es);
    L.hd = take(s->residual ? T * f * es : 0);
    // the dense branch's output where it is not combined in place: rounded, or sums in 32 bits (dense2_shared, dense2_split, with
    // either layout of the weights: no size depends on that).  What the sums take beyond the rounded output is room of its own, as much as
    // any smaller number of tokens wants: a workspace for a program's most tokens serves the others wherever one without the sums did
    size_t sums = (4 - es) * std::min(T, (size_t)kSharedTokens);
    if (T > 32) sums = std::max(sums, (4 * kLinearMaxSplit - es) * std::min(T, (size_t)kSplitTokens));
    L.dense = take(s->residual && plan.mfma ? T * d * es : 0);
    take(s->residual && plan.mfma ? sums * d : 0);
    L.partial = take(plan.ksplit_room > 1 ? (size_t)plan.ksplit_room * E * C * d * 4 : 0);
    L.total = off;
    return L;
}

template <typename T> inline T* at(void* ws, size_t off) { return reinterpret_cast<T*>(static_cast<char*>(ws) + off); }

int check_ws(const moe_shape_t* s, const void* ws, size_t ws_bytes) {
    if (!ws || !aligned16(ws) || ws_bytes < ws_layout(s).total) return MOE_ERR_WORKSPACE;
    return MOE_OK;
}

// The gate's share of the workspace: the leading regions of the layout (logits, split gate weights, histograms).
size_t gate_scratch_bytes(const moe_shape_t* s) { return ws_layout(s).expert_idx; }

// Scratch of moe_gate_noalloc: one array per GPU, inside the library's code object, so that the call needs no
// workspace from its caller and no allocation.  In host code the array's name is only a handle for
// hipGetSymbolAddress; kernels get the device address that call returns, looked up once per device.
constexpr size_t kStaticScratchBytes = 8u << 20;
constexpr int kMaxDevices = 64;
__device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes];
void* g_static_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MOE_ERR_HIP;
    if (!g_static_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch)) != hipSuccess || !p) return MOE_ERR_HIP;
        g_static_scratch_ptr[dev] = p;
    }
    *out = g_static_scratch_ptr[dev];
    return MOE_OK;
}

// gate logits: bf16 tokens go to the bf16 matrix cores when the shape allows, everything else to the fp32 ones.
// With MOE_FLAG_PACKED_GATE, Wg is the buffer moe_pack_gate wrote and no weight is split at call time.
int run_gate_logits(const moe_shape_t* s, const void* x, const float* Wg, const float* bg, float* logits, hipStream_t st) {
    const bool packed = s->flags & MOE_FLAG_PACKED_GATE;
    if (gate_on_bf16(s))
        return launch_gate_logits_bf16(x, packed ? nullptr : Wg, packed ? Wg : nullptr, bg, logits, s->T, s->d_model, s->E, st);
    return launch_gate_logits(x, s->dtype, Wg, bg, logits, s->T, s->d_model, s->E, st);
}

// the whole gate from tokens: logits (ST_LOGITS; with bf16 tokens and enough of them this kernel also does the
// top-k and the tile-local ranking) and the rest of the routing (ST_ROUTE)
int run_gate(const moe_shape_t* s, const void* x, const float* Wg, const float* bg, float* logits, int32_t* expert_idx,
             int32_t* slot_idx, float* gate_w, int32_t* rows, int32_t* slot_token, int32_t* order, void* ws,
             const WsLayout& L, bool profile, hipStream_t st) {
    int32_t* scratch = at<int32_t>(ws, L.hist);
    int rc;
    if (s->dtype == MOE_BF16 && gate_bf16_fused_supported(s->T, s->d_model, s->E)) {
        int tb = 0;
        const int32_t* hist = nullptr;
        const bool packed = s->flags & MOE_FLAG_PACKED_GATE;
        if (profile) prof_pre(ST_LOGITS, st);
        rc = launch_gate_bf16_fused(x, packed ? nullptr : Wg, packed ? Wg : nullptr, bg, logits, s->T, s->d_model, s->E,
                                    s->top_k, expert_idx, slot_idx, gate_w, at<void>(ws, L.wg_frags), scratch, &tb, &hist, st);
        if (profile) prof_mark(ST_LOGITS, st);
        if (rc != MOE_OK) return rc;
        if (profile) prof_pre(ST_ROUTE, st);
        rc = launch_route_finalize(s->T, s->E, s->top_k, s->capacity, tb, expert_idx, slot_idx, rows, slot_token, order,
                                   hist, st);
        if (profile) prof_mark(ST_ROUTE, st);
        return rc;
    }
    if (s->dtype == MOE_BF16 && gate_decode_supported(s->T, s->d_model, s->E)) {
        // decode: logits and the whole routing in one launch (counted under ST_LOGITS)
        const bool packed = s->flags & MOE_FLAG_PACKED_GATE;
        if (profile) prof_pre(ST_LOGITS, st);
        rc = launch_gate_decode(x, packed ? nullptr : Wg, packed ? Wg : nullptr, bg, logits, s->T, s->d_model, s->E,
                                s->top_k, s->capacity, expert_idx, slot_idx, gate_w, rows, slot_token, order,
                                at<uint64_t>(ws, L.flags), next_call_tag(), st);
        if (profile) prof_mark(ST_LOGITS, st);
        return rc;
    }
    if (profile) prof_pre(ST_LOGITS, st);
    if (!gate_on_bf16(s) && gate_logits_routes(s->T, s->E)) {
        int tb = 0;
        rc = launch_gate_logits_route(x, s->dtype, Wg, bg, logits, s->T, s->d_model, s->E, s->top_k, expert_idx, slot_idx, gate_w, scratch, &tb, st);
        if (profile) prof_mark(ST_LOGITS, st);
        if (rc != MOE_OK) return rc;
        if (profile) prof_pre(ST_ROUTE, st);
        rc = launch_route_finalize(s->T, s->E, s->top_k, s->capacity, tb, expert_idx, slot_idx, rows, slot_token, order, scratch, st);
        if (profile) prof_mark(ST_ROUTE, st);
        return rc;
    }
    rc = run_gate_logits(s, x, Wg, bg, logits, st);
    if (profile) prof_mark(ST_LOGITS, st);
    if (rc != MOE_OK) return rc;
    if (profile) prof_pre(ST_ROUTE, st);
    rc = launch_route(logits, s->T, s->E, s->top_k, s->capacity, expert_idx, slot_idx, gate_w, rows, slot_token, order,
                      scratch, st);
    if (profile) prof_mark(ST_ROUTE, st);
    return rc;
}

// First product of an fp32 FFN: h = gelu_tanh(rows of x W1 + b1), and the second one on its result
GemmArgs f32_expert_args(const moe_shape_t* s) {
    GemmArgs a{};
    a.max_rows = s->capacity; a.expect_rows = (int)(((long long)s->T * s->top_k + s->E - 1) / s->E); a.G = s->E; a.K = s->d_model; a.N = s->d_ffn;
    a.a_group_stride = s->capacity; a.o_group_stride = s->capacity;
    return a;
}
GemmArgs f32_dense_args(const moe_shape_t* s) {
    GemmArgs a{};
    a.fixed_rows = s->T; a.max_rows = s->T; a.G = 1; a.K = s->d_model; a.N = s->d_ffn;
    return a;
}
GemmArgs f32_second_args(const GemmArgs& a, const void* W2, const void* b2, void* out) {
    GemmArgs b = a;
    b.A = a.out; b.B = W2; b.bias = b2; b.out = out; b.row_map = nullptr; b.K = a.N; b.N = a.K;
    return b;
}

// The two GEMMs of the expert FFNs in fp32.  row_map == nullptr: rows are xin[e*C + r], else xin[row_map[e*C + r]]
// (dispatch fused in).  scatter_map == nullptr: rows of `out` are e*C + r, else the tokens' (top-1 combine fused in).
int run_expert_ffn_f32(const moe_shape_t* s, const void* xin, const int32_t* row_map, const int32_t* rows, const void* W1,
                       const void* b1, const void* W2, const void* b2, void* h, const int32_t* scatter_map,
                       const int32_t* slot_idx, const float* gate_w, void* out, hipStream_t st) {
    GemmArgs a = f32_expert_args(s);
    a.A = xin; a.B = W1; a.bias = b1; a.out = h; a.rows = rows; a.row_map = row_map;
    GemmArgs b = f32_second_args(a, W2, b2, out);
    b.scatter_map = scatter_map; b.T = s->T; b.gate_w = gate_w; b.slot_idx = slot_idx; b.top_k = s->top_k;
    const int epi = scatter_map ? EPI_SCATTER : EPI_STORE;
    prof_pre(ST_GEMM1, st);
    if (ffn_f32_fused(a)) {                   // counted under ST_GEMM1
        const int rc = launch_ffn_f32(a, b, epi, st);
        prof_mark(ST_GEMM1, st);
        return rc;
    }
    int rc = launch_gemm_f32(a, EPI_GELU, st);
    prof_mark(ST_GEMM1, st);
    if (rc != MOE_OK) return rc;
    prof_pre(ST_GEMM2, st);
    rc = launch_gemm_f32(b, epi, st);
    prof_mark(ST_GEMM2, st);
    return rc;
}

// Dense branch of an fp32 Residual-MoE layer, the combine fused into its second GEMM.
int run_dense_f32(const moe_shape_t* s, const void* x, const void* Wd1, const void* bd1, const void* Wd2, const void* bd2,
                  void* hd, const void* ye, const int32_t* expert_idx, const int32_t* slot_idx, const float* gate_w, void* out,
                  hipStream_t st) {
    GemmArgs a = f32_dense_args(s);
    a.A = x; a.B = Wd1; a.bias = bd1; a.out = hd;
    GemmArgs b = f32_second_args(a, Wd2, bd2, out);
    b.ye = ye; b.expert_idx = expert_idx; b.slot_idx = slot_idx; b.gate_w = gate_w; b.top_k = s->top_k; b.C = s->capacity;
    prof_pre(ST_DENSE1, st);
    if (ffn_f32_fused(a)) {                   // counted under ST_DENSE1
        const int rc = launch_ffn_f32(a, b, EPI_COMBINE, st);
        prof_mark(ST_DENSE1, st);
        return rc;
    }
    int rc = launch_gemm_f32(a, EPI_GELU, st);
    prof_mark(ST_DENSE1, st);
    if (rc != MOE_OK) return rc;
    prof_pre(ST_DENSE2, st);
    rc = launch_gemm_f32(b, EPI_COMBINE, st);
    prof_mark(ST_DENSE2, st);
    return rc;
}

inline const uint16_t* u16(const void* p) { return static_cast<const uint16_t*>(p); }
inline uint16_t* u16(void* p) { return static_cast<uint16_t*>(p); }

// Expert GEMM-1 on the MFMA kernels: h[e, r, :] = gelu_tanh(A_row(e, r) W1[e] + b1[e]).
// row_map == nullptr: A rows are xin[e*C + r]; otherwise xin[row_map[e*C + r]] (dispatch fused in).
WsGemmArgs expert_gemm1_args(const moe_shape_t* s, const FfnPlan& p, const void* xin, const int32_t* row_map,
                             const int32_t* rows, const int32_t* order, const void* W1, const void* b1, void* h) {
    WsGemmArgs a{};
    a.A = u16(xin); a.B = u16(W1); a.bias = u16(b1); a.rows = rows; a.order = order; a.row_map = row_map;
    a.packed = s->flags & MOE_FLAG_PACKED_WEIGHTS; a.slots = p.slots;
    a.max_rows = s->capacity; a.expect_rows = p.expect; a.map_stride = s->capacity; a.G = s->E; a.K = s->d_model; a.N = s->d_ffn;
    a.a_group_stride = s->capacity; a.out = u16(h); a.o_group_stride = s->capacity; a.ksplit = 1;
    return a;
}
// First product of the dense branch of Residual-MoE: hd = gelu_tanh(x Wd1 + bd1)
WsGemmArgs dense_gemm1_args(const moe_shape_t* s, const void* x, const void* Wd1, const void* bd1, void* hd) {
    WsGemmArgs a{};
    a.A = u16(x); a.B = u16(Wd1); a.bias = u16(bd1); a.fixed_rows = s->T; a.max_rows = s->T; a.G = 1;
    a.packed = s->flags & MOE_FLAG_PACKED_WEIGHTS;
    a.K = s->d_model; a.N = s->d_ffn; a.out = u16(hd); a.ksplit = 1;
    return a;
}

int run_expert_gemm1(const moe_shape_t* s, const FfnPlan& p, const void* xin, const int32_t* row_map,
                     const int32_t* rows, const int32_t* order, const void* W1, const void* b1, void* h,
                     hipStream_t st) {
    const WsGemmArgs a = expert_gemm1_args(s, p, xin, row_map, rows, order, W1, b1, h);
    prof_pre(ST_GEMM1, st);
    const int rc = p.nf1     ? launch_rows(a, nullptr, EPI_GELU, p.nf1, st)
                   : p.tiled1 ? launch_tgemm(a, EPI_GELU, st)
                             : launch_wsgemm(a, EPI_GELU, p.MT, p.NW1, p.NBUF, st);
    prof_mark(ST_GEMM1, st);
    return rc;
}

// Expert GEMM-2 on the MFMA kernel.  scatter == false: ye[e, r, :] = h[e, r, :] W2[e] + b2[e].
// scatter == true (top-1): out[token(e, r), :] = gate_w[token] * (...), rows of dropped tokens zeroed; with `add` (a decoder
// block) its rows are added.
int run_expert_gemm2(const moe_shape_t* s, const FfnPlan& p, const void* h, const int32_t* rows,
                     const int32_t* order, const void* W2, const void* b2, bool scatter, const int32_t* slot_token, const int32_t* slot_idx,
                     const float* gate_w, const uint16_t* add, void* dst, float* partial, hipStream_t st) {
    WsGemmArgs a{};
    a.A = u16(h); a.B = u16(W2); a.bias = u16(b2); a.rows = rows; a.row_map = nullptr;
    // The tiled kernel's tiles of this product are long (K = d_ffn) and few per CU: the busiest experts go first, so
    // that the short tiles of the light ones fill the end (the second list).  GEMM-1 and the streaming kernel keep
    // the list that alternates busy and light experts.
    a.order = order && p.tiled ? order + s->E + 1 : order;
    a.packed = s->flags & MOE_FLAG_PACKED_WEIGHTS; a.slots = p.slots;
    a.max_rows = s->capacity; a.expect_rows = p.expect; a.G = s->E; a.K = s->d_ffn; a.N = s->d_model;
    a.a_group_stride = s->capacity; a.out = u16(dst); a.o_group_stride = s->capacity; a.ksplit = p.ksplit2;
    a.scatter_map = slot_token; a.scatter_stride = s->capacity; a.zero_slot_idx = slot_idx; a.T = s->T;
    a.gate_w = gate_w; a.top_k = s->top_k; a.add = add;
    prof_pre(ST_GEMM2, st);
    if (p.ksplit2 == 1) {
        const int epi = scatter ? EPI_SCATTER : EPI_STORE;
        const int rc1 = p.nf2     ? launch_rows(a, nullptr, epi, p.nf2, st)
                        : p.tiled ? launch_tgemm(a, epi, st)
                                  : launch_wsgemm(a, epi, p.MT, p.NW2, p.NBUF, st);
        prof_mark(ST_GEMM2, st);
        return rc1;
    }
    a.partial = partial;
    a.partial_rows = (long long)s->E * s->capacity;
    a.split_tiles = order ? split_tiles(s, p) : 0;
    int rc = launch_wsgemm(a, EPI_PARTIAL, p.MT, p.NW2, p.NBUF, st);
    prof_mark(ST_GEMM2, st);
    if (rc != MOE_OK) return rc;
    SplitKReduceArgs r{};
    r.partial = partial; r.ksplit = p.ksplit2; r.G = s->E; r.N = s->d_model; r.group_stride = s->capacity;
    r.rows = rows; r.max_rows = s->capacity; r.bias = u16(b2); r.out = u16(dst); r.order = order; r.split_tiles = a.split_tiles;
    r.scatter_map = scatter ? slot_token : nullptr; r.gate_w = gate_w; r.top_k = s->top_k; r.add = add;
    r.zero_slot_idx = scatter ? slot_idx : nullptr; r.T = s->T;
    prof_pre(ST_REDUCE, st);
    rc = launch_splitk_reduce(r, st);
    prof_mark(ST_REDUCE, st);
    return rc;
}

// does the dense branch of so many tokens go to the tiled kernel (where the few-weights one does not take it)?
bool dense_tiled(const moe_shape_t* s) {
    return s->T > 64 && tgemm_supported(s->d_model, s->d_ffn) && tgemm_supported(s->d_ffn, s->d_model);
}
// does the dense branch's first product share the launch of the experts' in the few-weights kernel?
bool dense1_shared(const moe_shape_t* s, const FfnPlan& p) {
    return s->residual && p.nf1 && s->T <= 16 && rows_pick_dense(s->T, s->d_ffn, s->flags & MOE_FLAG_PACKED_WEIGHTS);
}

// First product of the dense branch: hd = gelu_tanh(x Wd1 + bd1)
int run_dense_first(const moe_shape_t* s, const void* x, const void* Wd1, const void* bd1, void* hd, hipStream_t st) {
    int MT, NW;
    const WsGemmArgs a = dense_gemm1_args(s, x, Wd1, bd1, hd);
    const int nf = rows_pick_dense(s->T, s->d_ffn, a.packed);
    wsgemm_pick_tile(s->T, 1, s->d_ffn, &MT, &NW);
    prof_pre(ST_DENSE1, st);
    const int rc = nf               ? launch_rows(a, nullptr, EPI_GELU, nf, st)
                   : dense_tiled(s) ? launch_tgemm(a, EPI_GELU, st)
                                    : launch_wsgemm(a, EPI_GELU, MT, NW, 2, st);
    prof_mark(ST_DENSE1, st);
    return rc;
}

// Dense branch of Residual-MoE on the MFMA kernels, with the combine fused into its second GEMM:
// out[t, :] = gelu_tanh(x[t] Wd1 + bd1) Wd2 + bd2 + sum_j keep_j g_j ye[e_j, slot_j, :] (+ add[t, :]).
// first_done: hd is there already (the first product shared a launch with the experts').
int run_dense_branch(const moe_shape_t* s, const void* x, const void* Wd1, const void* bd1, const void* Wd2,
                     const void* bd2, void* hd, bool first_done, const void* ye, const int32_t* expert_idx,
                     const int32_t* slot_idx, const float* gate_w, const uint16_t* add, void* out, hipStream_t st) {
    int MT, NW, rc = MOE_OK;
    if (!first_done) {
        rc = run_dense_first(s, x, Wd1, bd1, hd, st);
        if (rc != MOE_OK) return rc;
    }
    WsGemmArgs a = dense_gemm1_args(s, x, Wd1, bd1, hd);
    a.A = u16(hd); a.B = u16(Wd2); a.bias = u16(bd2); a.K = s->d_ffn; a.N = s->d_model; a.out = u16(out);
    a.ye = u16(ye); a.expert_idx = expert_idx; a.slot_idx = slot_idx; a.gate_w = gate_w; a.top_k = s->top_k;
    a.C = s->capacity; a.add = add;
    const int nf = rows_pick_dense(s->T, s->d_model, a.packed);
    wsgemm_pick_tile(s->T, 1, s->d_model, &MT, &NW);
    prof_pre(ST_DENSE2, st);
    rc = nf               ? launch_rows(a, nullptr, EPI_COMBINE, nf, st)
         : dense_tiled(s) ? launch_tgemm(a, EPI_COMBINE, st)
                          : launch_wsgemm(a, EPI_COMBINE, MT, NW, 2, st);
    prof_mark(ST_DENSE2, st);
    return rc;
}

// the second product of the FFN half that `a` is the first one of, on its output
WsGemmArgs second_half(WsGemmArgs a, const void* h, const void* W2, const void* b2, void* out) {
    a.A = u16(h); a.B = u16(W2); a.bias = u16(b2); a.row_map = nullptr; a.out = u16(out);
    const int K = a.K;
    a.K = a.N; a.N = K;
    return a;
}
// Do the experts' and the dense branch's second products share a launch?  Experts with room for at most 64 rows and shapes with
// an inner dimension off the 32-deep stages keep the combine inside the dense branch's product, which adds the experts' rows to
// unrounded sums.
bool residual_pairs(const moe_shape_t* s, const FfnPlan& p) {
    if (!p.tiled || s->capacity <= 64 || s->T <= 128 || s->d_model % 32 || s->d_ffn % 32) return false;
    return tgemm_pair_fusable(second_half(expert_gemm1_args(s, p, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr), nullptr, nullptr, nullptr, nullptr),
                              second_half(dense_gemm1_args(s, nullptr, nullptr, nullptr, nullptr), nullptr, nullptr, nullptr, nullptr));
}

// Can the layer's last kernel add rows to its results?  All can but the tiled ones.
bool layer_adds(const moe_shape_t* s, const FfnPlan& p) {
    if (!p.mfma) return false;
    if (!s->residual) return s->top_k == 2 || p.nf2 || !p.tiled;
    if (residual_pairs(s, p)) return false;
    return dense2_shared(s, p) || dense2_split(s) > 1 || rows_pick_dense(s->T, s->d_model, s->flags & MOE_FLAG_PACKED_WEIGHTS) || !dense_tiled(s);
}

// Residual-MoE with experts and dense branch both on the tiled kernel: the experts' and the dense branch's products of
// each FFN half share one launch (same inner and outer sizes), so that the second half, with only d_model columns,
// has more tiles and can use a larger one; the combine then is a kernel of its own on the two outputs.
// Returns MOE_ERR_UNSUPPORTED (nothing launched) when the pair does not fit that pattern.
int run_residual_paired(const moe_shape_t* s, const FfnPlan& p, const void* x, const int32_t* slot_token,
                        const int32_t* rows, const int32_t* order, const void* W1, const void* b1, const void* W2,
                        const void* b2, const void* Wd1, const void* bd1, const void* Wd2, const void* bd2, void* h,
                        void* hd, void* ye, void* dense_out, const int32_t* expert_idx, const int32_t* slot_idx,
                        const float* gate_w, void* out, hipStream_t st) {
    if (!residual_pairs(s, p)) return MOE_ERR_UNSUPPORTED;
    const WsGemmArgs e1 = expert_gemm1_args(s, p, x, slot_token, rows, order, W1, b1, h), d1 = dense_gemm1_args(s, x, Wd1, bd1, hd);
    const WsGemmArgs e2 = second_half(e1, h, W2, b2, ye), d2 = second_half(d1, hd, Wd2, bd2, dense_out);
    int rc;
    if (tgemm_pair_fusable(e1, d1)) {
        prof_pre(ST_GEMM1, st);
        rc = launch_tgemm_pair(e1, d1, EPI_GELU, st);
        prof_mark(ST_GEMM1, st);
    } else {                                  // the first halves each on the tile that suits them
        prof_pre(ST_GEMM1, st);
        rc = launch_tgemm(e1, EPI_GELU, st);
        prof_mark(ST_GEMM1, st);
        if (rc != MOE_OK) return rc;
        prof_pre(ST_DENSE1, st);
        rc = launch_tgemm(d1, EPI_GELU, st);
        prof_mark(ST_DENSE1, st);
    }
    if (rc != MOE_OK) return rc;
    prof_pre(ST_GEMM2, st);
    rc = launch_tgemm_pair(e2, d2, EPI_STORE, st);
    prof_mark(ST_GEMM2, st);
    if (rc != MOE_OK) return rc;
    prof_pre(ST_COMBINE, st);
    rc = launch_combine(ye, s->dtype, expert_idx, slot_idx, gate_w, dense_out, out, s->T, s->top_k, s->capacity,
                        s->d_model, st);
    prof_mark(ST_COMBINE, st);
    return rc;
}

}  // namespace

extern "C" {

size_t moe_workspace_bytes(const moe_shape_t* shape) {
    if (check_shape(shape) != MOE_OK) return 0;
    return ws_layout(shape).total;
}

const char* moe_status_string(int status) {
    switch (status) {
        case MOE_OK: return "ok";
        case MOE_ERR_INVALID_ARG: return "invalid argument";
        case MOE_ERR_UNSUPPORTED: return "unsupported shape";
        case MOE_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
        case MOE_ERR_HIP: return "HIP launch failed";
        case MOE_ERR_SCRATCH_LIMIT: return "shape needs more scratch than the no-allocation entry point holds";
        default: return "unknown status";
    }
}

const char* moe_version(void) { return "0.2"; }

size_t moe_packed_weights_bytes(int32_t G, int32_t K, int32_t N) {
    if (G < 1 || K < 8 || N < 8 || K % 8 || N % 8) return 0;
    return packed_weight_elems(G, K, N) * 2;
}

size_t moe_packed_gate_bytes(int32_t d_model, int32_t E) {
    if (d_model < 1 || E < 1) return 0;
    return gate_bf16_ws_bytes(d_model, E);            // 0 for shapes the bf16 gate kernel does not cover
}

int moe_pack_gate(int32_t d_model, int32_t E, const float* Wg, void* packed, void* stream) {
    if (d_model < 1 || E < 1 || !Wg || !packed || !aligned16(Wg) || !aligned16(packed)) return MOE_ERR_INVALID_ARG;
    return launch_pack_gate(Wg, packed, d_model, E, static_cast<hipStream_t>(stream));
}

int moe_pack_weights(int32_t G, int32_t K, int32_t N, const void* W, void* packed, void* stream) {
    if (G < 1 || K < 8 || N < 8 || !W || !packed || !aligned16(W) || !aligned16(packed)) return MOE_ERR_INVALID_ARG;
    if (K % 8 || N % 8) return MOE_ERR_UNSUPPORTED;
    return launch_pack_weights(u16(W), u16(packed), G, K, N, static_cast<hipStream_t>(stream));
}

// argument checks shared by moe_gate and moe_gate_noalloc (everything but the scratch memory)
static int check_gate_args(const moe_shape_t* shape, const void* x, const float* Wg, const float* bg, float* logits,
                           int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* expert_rows,
                           int32_t* slot_token) {
    const int rc = check_shape(shape);
    if (rc != MOE_OK) return rc;
    if (!expert_idx || !slot_idx || !gate_w || !expert_rows || !slot_token) return MOE_ERR_INVALID_ARG;
    if (!x && !logits) return MOE_ERR_INVALID_ARG;
    if (x && !Wg) return MOE_ERR_INVALID_ARG;
    const void* ptrs[] = {x, Wg, bg, logits, expert_idx, slot_idx, gate_w, expert_rows, slot_token};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return MOE_ERR_INVALID_ARG;
    return MOE_OK;
}

// the gate on checked arguments; `ws` holds at least gate_scratch_bytes(shape) bytes
static int gate_checked(const moe_shape_t* shape, const void* x, const float* Wg, const float* bg, float* logits,
                        int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* expert_rows,
                        int32_t* slot_token, void* ws, hipStream_t st) {
    const WsLayout L = ws_layout(shape);
    float* lg = logits ? logits : at<float>(ws, L.logits);
    if (x)
        return run_gate(shape, x, Wg, bg, lg, expert_idx, slot_idx, gate_w, expert_rows, slot_token, nullptr, ws, L, false, st);
    return launch_route(lg, shape->T, shape->E, shape->top_k, shape->capacity, expert_idx, slot_idx, gate_w,
                        expert_rows, slot_token, nullptr, at<int32_t>(ws, L.hist), st);
}

int moe_gate(const moe_shape_t* shape, const void* x, const float* Wg, const float* bg, float* logits,
             int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* expert_rows, int32_t* slot_token,
             void* ws, size_t ws_bytes, void* stream) {
    int rc = check_gate_args(shape, x, Wg, bg, logits, expert_idx, slot_idx, gate_w, expert_rows, slot_token);
    if (rc != MOE_OK) return rc;
    rc = check_ws(shape, ws, ws_bytes);
    if (rc != MOE_OK) return rc;
    return gate_checked(shape, x, Wg, bg, logits, expert_idx, slot_idx, gate_w, expert_rows, slot_token, ws,
                        static_cast<hipStream_t>(stream));
}

size_t moe_gate_noalloc_max_bytes(void) { return kStaticScratchBytes; }

size_t moe_gate_noalloc_bytes(const moe_shape_t* shape) {
    if (check_shape(shape) != MOE_OK) return 0;
    return gate_scratch_bytes(shape);
}

int moe_gate_noalloc(const moe_shape_t* shape, const void* x, const float* Wg, const float* bg, float* logits,
                     int32_t* expert_idx, int32_t* slot_idx, float* gate_w, int32_t* expert_rows, int32_t* slot_token,
                     void* stream) {
    int rc = check_gate_args(shape, x, Wg, bg, logits, expert_idx, slot_idx, gate_w, expert_rows, slot_token);
    if (rc != MOE_OK) return rc;
    if (gate_scratch_bytes(shape) > kStaticScratchBytes) return MOE_ERR_SCRATCH_LIMIT;
    void* scratch = nullptr;
    rc = static_scratch(&scratch);
    if (rc != MOE_OK) return rc;
    return gate_checked(shape, x, Wg, bg, logits, expert_idx, slot_idx, gate_w, expert_rows, slot_token, scratch,
                        static_cast<hipStream_t>(stream));
}

int moe_dispatch(const moe_shape_t* shape, const void* x, const int32_t* slot_token, const int32_t* expert_rows,
                 void* xe, void* stream) {
    int rc = check_shape(shape);
    if (rc != MOE_OK) return rc;
    if (!x || !slot_token || !expert_rows || !xe) return MOE_ERR_INVALID_ARG;
    if (!aligned16(x) || !aligned16(slot_token) || !aligned16(expert_rows) || !aligned16(xe)) return MOE_ERR_INVALID_ARG;
    return launch_dispatch(x, shape->dtype, slot_token, expert_rows, xe, shape->E, shape->capacity, shape->d_model,
                           static_cast<hipStream_t>(stream));
}

int moe_expert_ffn(const moe_shape_t* shape, const void* xe, const int32_t* expert_rows, const void* W1,
                   const void* b1, const void* W2, const void* b2, void* ye, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_shape(shape);
    if (rc != MOE_OK) return rc;
    if (!xe || !expert_rows || !W1 || !W2 || !ye) return MOE_ERR_INVALID_ARG;
    const void* ptrs[] = {xe, expert_rows, W1, b1, W2, b2, ye};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return MOE_ERR_INVALID_ARG;
    rc = check_ws(shape, ws, ws_bytes);
    if (rc != MOE_OK) return rc;
    const WsLayout L = ws_layout(shape);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const FfnPlan plan = plan_ffn(shape);
    if (!plan.mfma)
        return run_expert_ffn_f32(shape, xe, nullptr, expert_rows, W1, b1, W2, b2, at<void>(ws, L.h), nullptr, nullptr, nullptr,
                                  ye, st);
    int32_t* order = at<int32_t>(ws, L.order);
    rc = launch_expert_order(expert_rows, shape->E, shape->capacity, order, st);
    if (rc != MOE_OK) return rc;
    rc = run_expert_gemm1(shape, plan, xe, nullptr, expert_rows, order, W1, b1, at<void>(ws, L.h), st);
    if (rc != MOE_OK) return rc;
    return run_expert_gemm2(shape, plan, at<void>(ws, L.h), expert_rows, order, W2, b2, false, nullptr, nullptr, nullptr, nullptr, ye,
                            at<float>(ws, L.partial), st);
}

int moe_expert_ffn_slice(const moe_shape_t* shape, const void* xe, const int32_t* expert_rows, const void* W1s,
                         const void* b1s, const void* W2s, float* ye_partial, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_shape(shape);
    if (rc != MOE_OK) return rc;
    if (shape->dtype != MOE_BF16) return MOE_ERR_UNSUPPORTED;
    if (!xe || !expert_rows || !W1s || !W2s || !ye_partial) return MOE_ERR_INVALID_ARG;
    const void* ptrs[] = {xe, expert_rows, W1s, b1s, W2s, ye_partial};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return MOE_ERR_INVALID_ARG;
    rc = check_ws(shape, ws, ws_bytes);
    if (rc != MOE_OK) return rc;
    const WsLayout L = ws_layout(shape);
    hipStream_t st = static_cast<hipStream_t>(stream);
    FfnPlan plan = plan_ffn(shape);
    plan.ksplit2 = 1;                                  // the slice itself is the split of the inner dimension
    int32_t* order = at<int32_t>(ws, L.order);
    rc = launch_expert_order(expert_rows, shape->E, shape->capacity, order, st);
    if (rc != MOE_OK) return rc;
    rc = run_expert_gemm1(shape, plan, xe, nullptr, expert_rows, order, W1s, b1s, at<void>(ws, L.h), st);
    if (rc != MOE_OK) return rc;
    WsGemmArgs a{};
    a.A = at<uint16_t>(ws, L.h); a.B = u16(W2s); a.rows = expert_rows; a.order = order;
    a.packed = shape->flags & MOE_FLAG_PACKED_WEIGHTS;
    a.max_rows = shape->capacity; a.expect_rows = plan.expect; a.G = shape->E; a.K = shape->d_ffn; a.N = shape->d_model;
    a.a_group_stride = shape->capacity; a.o_group_stride = shape->capacity; a.ksplit = 1;
    a.partial = ye_partial; a.partial_rows = (long long)shape->E * shape->capacity;
    return plan.tiled ? launch_tgemm(a, EPI_PARTIAL, st) : launch_wsgemm(a, EPI_PARTIAL, plan.MT, plan.NW2, plan.NBUF, st);
}

int moe_expert_ffn_slice_reduce(const moe_shape_t* shape, int32_t n_slices, const float* ye_partials,
                                const int32_t* expert_rows, const void* b2, void* ye, void* stream) {
    int rc = check_shape(shape);
    if (rc != MOE_OK) return rc;
    if (shape->dtype != MOE_BF16) return MOE_ERR_UNSUPPORTED;
    if (n_slices < 1 || n_slices > 64 || !ye_partials || !expert_rows || !ye) return MOE_ERR_INVALID_ARG;
    if (!aligned16(ye_partials) || !aligned16(expert_rows) || !aligned16(ye) || (b2 && !aligned16(b2)))
        return MOE_ERR_INVALID_ARG;
    SplitKReduceArgs r{};
    r.partial = ye_partials; r.ksplit = n_slices; r.G = shape->E; r.N = shape->d_model; r.group_stride = shape->capacity;
    r.rows = expert_rows; r.max_rows = shape->capacity; r.bias = u16(b2); r.out = u16(ye); r.top_k = shape->top_k;
    r.T = shape->T;
    return launch_splitk_reduce(r, static_cast<hipStream_t>(stream));
}

int moe_combine(const moe_shape_t* shape, const void* ye, const int32_t* expert_idx, const int32_t* slot_idx,
                const float* gate_w, const void* addend, void* out, void* stream) {
    int rc = check_shape(shape);
    if (rc != MOE_OK) return rc;
    if (!ye || !expert_idx || !slot_idx || !gate_w || !out) return MOE_ERR_INVALID_ARG;
    const void* ptrs[] = {ye, expert_idx, slot_idx, gate_w, addend, out};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return MOE_ERR_INVALID_ARG;
    return launch_combine(ye, shape->dtype, expert_idx, slot_idx, gate_w, addend, out, shape->T, shape->top_k,
                          shape->capacity, shape->d_model, static_cast<hipStream_t>(stream));
}

static int layer_forward_checked(const moe_shape_t* shape, const void* x, const float* Wg, const float* bg, const void* W1,
                      const void* b1, const void* W2, const void* b2, const void* Wd1, const void* bd1, const void* Wd2,
                      const void* bd2, void* out, float* logits_out, int32_t* expert_idx_out, int32_t* slot_idx_out,
                      float* gate_w_out, int32_t* expert_rows_out, int32_t* slot_token_out, void* ws, size_t ws_bytes,
                      const uint16_t* add, void* stream) {
    int rc = check_shape(shape);
    if (rc != MOE_OK) return rc;
    if (!x || !Wg || !W1 || !W2 || !out) return MOE_ERR_INVALID_ARG;
    if (shape->residual && (!Wd1 || !Wd2)) return MOE_ERR_INVALID_ARG;
    if (!shape->residual && (Wd1 || Wd2 || bd1 || bd2)) return MOE_ERR_INVALID_ARG;
    const void* ptrs[] = {x, Wg, bg, W1, b1, W2, b2, Wd1, bd1, Wd2, bd2, out, logits_out, expert_idx_out,
                          slot_idx_out, gate_w_out, expert_rows_out, slot_token_out};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return MOE_ERR_INVALID_ARG;
    rc = check_ws(shape, ws, ws_bytes);
    if (rc != MOE_OK) return rc;

    const WsLayout L = ws_layout(shape);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int T = shape->T, d = shape->d_model, f = shape->d_ffn, E = shape->E, k = shape->top_k, C = shape->capacity;
    const int dt = shape->dtype;

    float* logits = logits_out ? logits_out : at<float>(ws, L.logits);
    int32_t* expert_idx = expert_idx_out ? expert_idx_out : at<int32_t>(ws, L.expert_idx);
    int32_t* slot_idx = slot_idx_out ? slot_idx_out : at<int32_t>(ws, L.slot_idx);
    float* gate_w = gate_w_out ? gate_w_out : at<float>(ws, L.gate_w);
    int32_t* rows = expert_rows_out ? expert_rows_out : at<int32_t>(ws, L.rows);
    int32_t* slot_token = slot_token_out ? slot_token_out : at<int32_t>(ws, L.slot_token);

    prof_begin(st);
    int32_t* order = at<int32_t>(ws, L.order);
    rc = run_gate(shape, x, Wg, bg, logits, expert_idx, slot_idx, gate_w, rows, slot_token, order, ws, L, true, st);
    if (rc != MOE_OK) return rc;
    FfnPlan plan = plan_ffn(shape);
    plan.slots = (int)((long long)T * k < E ? (long long)T * k : E);
    if (!plan.mfma) {
        // fp32 layer: rows gathered inside GEMM-1; combine inside GEMM-2 (top-1), the dense branch's second GEMM
        // (residual) or, for top-2, a kernel of its own
        const bool scatter = k == 1 && !shape->residual;
        void* ye = at<void>(ws, L.ye);
        rc = run_expert_ffn_f32(shape, x, slot_token, rows, W1, b1, W2, b2, at<void>(ws, L.h), scatter ? slot_token : nullptr,
                                slot_idx, gate_w, scatter ? out : ye, st);
        if (rc != MOE_OK || scatter) return rc;
        if (shape->residual)
            return run_dense_f32(shape, x, Wd1, bd1, Wd2, bd2, at<void>(ws, L.hd), ye, expert_idx, slot_idx, gate_w, out, st);
        prof_pre(ST_COMBINE, st);
        rc = launch_combine(ye, dt, expert_idx, slot_idx, gate_w, nullptr, out, T, k, C, d, st);
        prof_mark(ST_COMBINE, st);
        return rc;
    }

    if (shape->residual) {
        rc = run_residual_paired(shape, plan, x, slot_token, rows, order, W1, b1, W2, b2, Wd1, bd1, Wd2, bd2,
                                 at<void>(ws, L.h), at<void>(ws, L.hd), at<void>(ws, L.ye), at<void>(ws, L.dense),
                                 expert_idx, slot_idx, gate_w, out, st);
        if (rc != MOE_ERR_UNSUPPORTED) return rc;
    }
    // bf16: dispatch is fused into GEMM-1 (rows gathered through slot_token) ...
    bool dense1_done = false;
    if (dense1_shared(shape, plan)) {
        // ... which takes the dense branch's first product along when both read little but weights
        const WsGemmArgs d1 = dense_gemm1_args(shape, x, Wd1, bd1, at<void>(ws, L.hd));
        prof_pre(ST_GEMM1, st);
        rc = launch_rows(expert_gemm1_args(shape, plan, x, slot_token, rows, order, W1, b1, at<void>(ws, L.h)), &d1, EPI_GELU,
                         plan.nf1, st);
        prof_mark(ST_GEMM1, st);
        dense1_done = true;
    } else {
        rc = run_expert_gemm1(shape, plan, x, slot_token, rows, order, W1, b1, at<void>(ws, L.h), st);
    }
    if (rc != MOE_OK) return rc;
    // ... and, for top-1 Standard-MoE, combine into GEMM-2 (scale by the gate weight, write the token's row)
    if (k == 1 && !shape->residual)
        return run_expert_gemm2(shape, plan, at<void>(ws, L.h), rows, order, W2, b2, true, slot_token, slot_idx, gate_w, add, out,
                                at<float>(ws, L.partial), st);
    if (dense2_shared(shape, plan)) {
        if (!dense1_done) {
            rc = run_dense_first(shape, x, Wd1, bd1, at<void>(ws, L.hd), st);
            if (rc != MOE_OK) return rc;
        }
        WsGemmArgs d2 = second_half(dense_gemm1_args(shape, nullptr, nullptr, nullptr, nullptr), at<void>(ws, L.hd), Wd2, bd2, nullptr);
        d2.partial = at<float>(ws, L.dense);
        const WsGemmArgs e2 = second_half(expert_gemm1_args(shape, plan, nullptr, nullptr, rows, order, nullptr, nullptr, nullptr),
                                          at<void>(ws, L.h), W2, b2, at<void>(ws, L.ye));
        prof_pre(ST_GEMM2, st);
        rc = launch_rows(d2, &e2, EPI_STORE, plan.nf2, st);      // the dense branch's work-groups, with more rows, first
        prof_mark(ST_GEMM2, st);
        if (rc != MOE_OK) return rc;
        prof_pre(ST_COMBINE, st);
        rc = launch_combine(at<void>(ws, L.ye), dt, expert_idx, slot_idx, gate_w, add, out, T, k, C, d, st, PartSums{at<float>(ws, L.dense), 1, nullptr});
        prof_mark(ST_COMBINE, st);
        return rc;
    }
    rc = run_expert_gemm2(shape, plan, at<void>(ws, L.h), rows, order, W2, b2, false, nullptr, nullptr, nullptr, nullptr,
                          at<void>(ws, L.ye), at<float>(ws, L.partial), st);
    if (rc != MOE_OK) return rc;
    if (shape->residual && dense2_split(shape) > 1) {
        if (!dense1_done) {
            rc = run_dense_first(shape, x, Wd1, bd1, at<void>(ws, L.hd), st);
            if (rc != MOE_OK) return rc;
        }
        WsGemmArgs d2 = second_half(dense_gemm1_args(shape, nullptr, nullptr, nullptr, nullptr), at<void>(ws, L.hd), Wd2, nullptr, nullptr);
        d2.ksplit = dense2_split(shape); d2.partial = at<float>(ws, L.dense); d2.partial_rows = T; d2.o_group_stride = T;
        int MT, NW;
        wsgemm_pick_tile(T, 1, d, &MT, &NW);
        prof_pre(ST_DENSE2, st);
        rc = launch_wsgemm(d2, EPI_PARTIAL, MT, NW, 2, st);
        prof_mark(ST_DENSE2, st);
        if (rc != MOE_OK) return rc;
        prof_pre(ST_COMBINE, st);
        rc = launch_combine(at<void>(ws, L.ye), dt, expert_idx, slot_idx, gate_w, add, out, T, k, C, d, st, PartSums{d2.partial, d2.ksplit, u16(bd2)});
        prof_mark(ST_COMBINE, st);
        return rc;
    }
    if (shape->residual)
        return run_dense_branch(shape, x, Wd1, bd1, Wd2, bd2, at<void>(ws, L.hd), dense1_done, at<void>(ws, L.ye),
                                expert_idx, slot_idx, gate_w, add, out, st);
    prof_pre(ST_COMBINE, st);
    rc = launch_combine(at<void>(ws, L.ye), dt, expert_idx, slot_idx, gate_w, add, out, T, k, C, d, st);
    prof_mark(ST_COMBINE, st);
    return rc;
}

int moe_layer_forward(const moe_shape_t* shape, const void* x, const float* Wg, const float* bg, const void* W1,
                      const void* b1, const void* W2, const void* b2, const void* Wd1, const void* bd1, const void* Wd2,
                      const void* bd2, void* out, float* logits_out, int32_t* expert_idx_out, int32_t* slot_idx_out,
                      float* gate_w_out, int32_t* expert_rows_out, int32_t* slot_token_out, void* ws, size_t ws_bytes,
                      void* stream) {
    const int rc = layer_forward_checked(shape, x, Wg, bg, W1, b1, W2, b2, Wd1, bd1, Wd2, bd2, out, logits_out,
                                         expert_idx_out, slot_idx_out, gate_w_out, expert_rows_out, slot_token_out, ws,
                                         ws_bytes, nullptr, stream);
    g_prof.cur = -1;       // stage events belong to this call only: a later moe_expert_ffn must not add to them
    return rc;
}

// Which kernel each product of a moe_layer_forward call takes, from the shape alone; for the tests of the dispatch, not
// part of the interface (moe.h does not declare it).  kernels: expert GEMM-1, expert GEMM-2, dense GEMM-1, dense GEMM-2, each
// 0 = none; fp32: F32Kernel; bf16: 1..4 = few-weights kernel with that many 16-column fragments, 100 S + rows = streaming kernel with tiles of that
// many rows and K split S ways, beyond that a tiled kernel (tgemm_code).
// shared: do the experts' and the dense product of the first / second half run in one launch, the second one's dense results rounded
// for the combine?  Dense GEMM-2 < 0: in the experts' launch of the few-weights kernel, its sums unrounded.
int moe_test_plan(const moe_shape_t* shape, int32_t kernels[4], int32_t shared[2]) {
    const int rc = check_shape(shape);
    if (rc != MOE_OK) return rc;
    const FfnPlan p = plan_ffn(shape);
    if (!p.mfma && shape->dtype != MOE_F32) return MOE_ERR_UNSUPPORTED;
    for (int i = 0; i < 4; ++i) kernels[i] = 0;
    shared[0] = shared[1] = 0;
    if (!p.mfma) {
        for (int i = 0; i < (shape->residual ? 4 : 2); i += 2) {
            const GemmArgs a = i ? f32_dense_args(shape) : f32_expert_args(shape);
            const bool fused = ffn_f32_fused(a);
            kernels[i] = fused ? F32_FFN : f32_kernel(a);
            kernels[i + 1] = fused ? F32_FFN : f32_kernel(f32_second_args(a, nullptr, nullptr, nullptr));
        }
        return MOE_OK;
    }
    const WsGemmArgs e1 = expert_gemm1_args(shape, p, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
    const WsGemmArgs d1 = dense_gemm1_args(shape, nullptr, nullptr, nullptr, nullptr);
    const WsGemmArgs e2 = second_half(e1, nullptr, nullptr, nullptr, nullptr), d2 = second_half(d1, nullptr, nullptr, nullptr, nullptr);
    if (shape->residual && residual_pairs(shape, p)) {
        shared[0] = tgemm_pair_fusable(e1, d1);
        shared[1] = 1;
        kernels[0] = tgemm_code(e1, shared[0] ? &d1 : nullptr, EPI_GELU);
        kernels[2] = shared[0] ? kernels[0] : tgemm_code(d1, nullptr, EPI_GELU);
        kernels[1] = kernels[3] = tgemm_code(e2, &d2, EPI_STORE);
        return MOE_OK;
    }
    kernels[0] = p.nf1 ? p.nf1 : p.tiled1 ? tgemm_code(e1, nullptr, EPI_GELU) : 100 + p.MT;
    kernels[1] = p.nf2 ? p.nf2 : p.tiled ? tgemm_code(e2, nullptr, shape->top_k == 1 && !shape->residual ? EPI_SCATTER : EPI_STORE) : 100 * p.ksplit2 + p.MT;
    if (!shape->residual) return MOE_OK;
    shared[0] = dense1_shared(shape, p);
    const bool sums = dense2_shared(shape, p);
    for (int i = 0; i < 2; ++i) {
        const WsGemmArgs& a = i ? d2 : d1;
        const int nf = rows_pick_dense(shape->T, a.N, a.packed);
        int MT, NW;
        wsgemm_pick_tile(shape->T, 1, a.N, &MT, &NW);
        const int ks = i ? dense2_split(shape) : 1;
        kernels[2 + i] = i && sums ? -p.nf2 : shared[i] ? p.nf1 : ks > 1 ? 100 * ks + MT : nf ? nf : dense_tiled(shape) ? tgemm_code(a, nullptr, i ? EPI_COMBINE : EPI_GELU) : 100 + MT;
    }
    return MOE_OK;
}

// ---- one decode step of a whole decoder block ---------------------------------------------------------------------
namespace {

struct BlockLayout {
    size_t qkv, attn, proj, x1, xn, moe_out, attn_partial, lin_partial, moe_ws, total;
};

BlockLayout block_layout(const moe_shape_t* s, const moe_block_shape_t* b) {
    BlockLayout L{};
    const size_t T = s->T, d = s->d_model;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += align_up(bytes); return o; };
    L.qkv = take(T * 3 * d * 2);
    L.attn = take(T * d * 2);
    L.proj = take(T * d * 2);
    L.x1 = take(T * d * 2);
    L.xn = take(T * d * 2);
    L.moe_out = take(T * d * 2);
    L.attn_partial = take(attn_partial_floats(s->T, b->n_heads, s->d_model / b->n_heads, b->max_len) * 4);
    L.lin_partial = take((size_t)kLinearMaxSplit * T * 3 * d * 4);
    L.moe_ws = take(ws_layout(s).total);
    L.total = off;
    return L;
}

int check_block_shape(const moe_shape_t* s, const moe_block_shape_t* b) {
    const int rc = check_shape(s);
    if (rc != MOE_OK) return rc;
    if (!b || b->n_heads < 1 || b->max_len < 1) return MOE_ERR_INVALID_ARG;
    if (s->dtype != MOE_BF16) return MOE_ERR_UNSUPPORTED;
    if (!attn_supported(s->d_model, b->n_heads)) return MOE_ERR_UNSUPPORTED;
    if ((long long)s->T * b->n_heads >= (1ll << 31) || b->max_len > (1 << 24)) return MOE_ERR_UNSUPPORTED;
    return MOE_OK;
}

// out[T, N] = x[T, K] W[K, N] + bias on the weight-streaming kernel (a decode step has few rows: the product is a
// read of W); with few output columns the inner dimension is split over more waves and summed in a fixed order: here, or
// (split_out given and more than 1) by whoever reads `partial` next
int run_linear(const uint16_t* x, const uint16_t* W, const uint16_t* bias, uint16_t* out, int T, int K, int N,
               float* partial, int* split_out, hipStream_t st) {
    if (split_out) *split_out = 1;
    WsGemmArgs a{};
    a.A = x; a.B = W; a.bias = bias; a.fixed_rows = T; a.max_rows = T; a.G = 1; a.K = K; a.N = N; a.out = out;
    a.o_group_stride = T; a.a_group_stride = T; a.ksplit = 1;
    if (T <= 32) return launch_rows(a, nullptr, EPI_STORE, 2, st);   // 64 rows: two launches 151 us, one 158 (d = 1024)
    int MT, NW;
    wsgemm_pick_tile(T, 1, N, &MT, &NW);
    const long long waves = (long long)((N + 127) / 128) * ((T + MT - 1) / MT);
    const int chunks = (K + wsgemm_chunk_k(MT) - 1) / wsgemm_chunk_k(MT);
    long long ks = waves < 1024 ? (2048 + waves - 1) / waves : 1;
    if (ks > kLinearMaxSplit) ks = kLinearMaxSplit;
    if (ks > chunks) ks = chunks;
    if (ks <= 1) return launch_wsgemm(a, EPI_STORE, MT, NW, 2, st);
    a.ksplit = (int)ks; a.partial = partial; a.partial_rows = T;
    int rc = launch_wsgemm(a, EPI_PARTIAL, MT, NW, 2, st);
    if (rc != MOE_OK) return rc;
    if (split_out) {
        *split_out = (int)ks;
        return MOE_OK;
    }
    SplitKReduceArgs r{};
    r.partial = partial; r.ksplit = (int)ks; r.G = 1; r.N = N; r.group_stride = T; r.rows = nullptr; r.max_rows = T;
    r.bias = bias; r.out = out; r.top_k = 1; r.T = T;
    return launch_splitk_reduce(r, st);
}

}  // namespace

size_t moe_decode_block_workspace_bytes(const moe_shape_t* shape, const moe_block_shape_t* block) {
    if (check_block_shape(shape, block) != MOE_OK) return 0;
    return block_layout(shape, block).total;
}

int moe_decode_block_forward(const moe_shape_t* shape, const moe_block_shape_t* block, const moe_block_weights_t* w,
                             const void* x, void* k_cache, void* v_cache, const int32_t* pos, void* out, void* x1_out,
                             void* moe_in_out, float* logits_out, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_block_shape(shape, block);
    if (rc != MOE_OK) return rc;
    if (!w || !x || !k_cache || !v_cache || !pos || !out) return MOE_ERR_INVALID_ARG;
    if (!w->ln1_gamma || !w->ln1_beta || !w->Wqkv || !w->Wo || !w->ln2_gamma || !w->ln2_beta || !w->Wg || !w->W1 || !w->W2)
        return MOE_ERR_INVALID_ARG;
    if (shape->residual && (!w->Wd1 || !w->Wd2)) return MOE_ERR_INVALID_ARG;
    if (!shape->residual && (w->Wd1 || w->Wd2 || w->bd1 || w->bd2)) return MOE_ERR_INVALID_ARG;
    const void* ptrs[] = {x, k_cache, v_cache, pos, out, x1_out, moe_in_out, logits_out, w->ln1_gamma, w->ln1_beta, w->Wqkv,
                          w->bqkv, w->Wo, w->bo, w->ln2_gamma, w->ln2_beta, w->Wg, w->bg, w->W1, w->b1, w->W2, w->b2,
                          w->Wd1, w->bd1, w->Wd2, w->bd2};
    for (const void* p : ptrs)
        if (p && !aligned16(p)) return MOE_ERR_INVALID_ARG;
    const BlockLayout L = block_layout(shape, block);
    if (!ws || !aligned16(ws) || ws_bytes < L.total) return MOE_ERR_WORKSPACE;

    hipStream_t st = static_cast<hipStream_t>(stream);
    const int T = shape->T, d = shape->d_model, H = block->n_heads, dh = d / H;
    const float eps = 1e-5f;
    uint16_t* qkv = at<uint16_t>(ws, L.qkv);
    uint16_t* attn = at<uint16_t>(ws, L.attn);
    uint16_t* proj = at<uint16_t>(ws, L.proj);
    uint16_t* x1 = x1_out ? u16(x1_out) : at<uint16_t>(ws, L.x1);
    uint16_t* xn = at<uint16_t>(ws, L.xn);
    uint16_t* moe_in = moe_in_out ? u16(moe_in_out) : xn;
    uint16_t* moe_out = at<uint16_t>(ws, L.moe_out);
    float* lin_partial = at<float>(ws, L.lin_partial);

    // a = LayerNorm(x); qkv = a Wqkv + bqkv
    rc = launch_add_layernorm(u16(x), AddedRows{}, w->ln1_gamma, w->ln1_beta, nullptr, xn, T, d, eps, st);
    if (rc != MOE_OK) return rc;
    rc = run_linear(xn, u16(w->Wqkv), u16(w->bqkv), qkv, T, d, 3 * d, lin_partial, nullptr, st);
    if (rc != MOE_OK) return rc;
    // the new token over its sequence's cache (its own key/value rows join the cache)
    rc = launch_attn_decode(qkv, u16(k_cache), u16(v_cache), pos, at<float>(ws, L.attn_partial), attn, T, H, dh,
                            block->max_len, st);
    if (rc != MOE_OK) return rc;
    int split = 1;
    rc = run_linear(attn, u16(w->Wo), u16(w->bo), proj, T, d, d, lin_partial, add_layernorm_sums(d) ? &split : nullptr, st);
    if (rc != MOE_OK) return rc;
    // x1 = x + attention; the MoE layer sees LayerNorm(x1)
    const AddedRows projected = split > 1 ? AddedRows{nullptr, PartSums{lin_partial, split, u16(w->bo)}} : AddedRows{proj, PartSums{}};
    rc = launch_add_layernorm(u16(x), projected, w->ln2_gamma, w->ln2_beta, x1, moe_in, T, d, eps, st);
    if (rc != MOE_OK) return rc;
    // out = x1 + MoE: in the layer's last kernel or behind it
    if (!layer_adds(shape, plan_ffn(shape))) {
        rc = layer_forward_checked(shape, moe_in, w->Wg, w->bg, w->W1, w->b1, w->W2, w->b2, w->Wd1, w->bd1, w->Wd2, w->bd2,
                                   moe_out, logits_out, nullptr, nullptr, nullptr, nullptr, nullptr,
                                   at<void>(ws, L.moe_ws), ws_layout(shape).total, nullptr, stream);
        g_prof.cur = -1;
        if (rc != MOE_OK) return rc;
        return launch_add_rows(x1, moe_out, u16(out), (long long)T * d, st);
    }
    rc = layer_forward_checked(shape, moe_in, w->Wg, w->bg, w->W1, w->b1, w->W2, w->b2, w->Wd1, w->bd1, w->Wd2, w->bd2,
                               out, logits_out, nullptr, nullptr, nullptr, nullptr, nullptr,
                               at<void>(ws, L.moe_ws), ws_layout(shape).total, x1, stream);
    g_prof.cur = -1;
    return rc;
}

int moe_profile_enable(int max_calls) {
    for (hipEvent_t e : g_prof.ev) (void)hipEventDestroy(e);
    g_prof.ev.clear(); g_prof.stage.clear(); g_prof.nmarks.clear();
    g_prof.max_calls = 0; g_prof.calls = 0; g_prof.cur = -1; g_prof.seen = 0;
    if (max_calls <= 0) return MOE_OK;
    if (max_calls > 4096) return MOE_ERR_INVALID_ARG;
    const size_t n = (size_t)max_calls * kMarks;
    g_prof.ev.resize(n);
    for (size_t i = 0; i < n; ++i)
        if (hipEventCreate(&g_prof.ev[i]) != hipSuccess) { g_prof.ev.resize(i); moe_profile_enable(0); return MOE_ERR_HIP; }
    g_prof.stage.assign(n, -1);
    g_prof.nmarks.assign(max_calls, 0);
    g_prof.max_calls = max_calls;
    return MOE_OK;
}

int moe_profile_select(unsigned stage_mask) {
    g_prof.mask = stage_mask;
    return MOE_OK;
}

int moe_profile_stride(int every_nth_call) {
    if (every_nth_call < 1) return MOE_ERR_INVALID_ARG;
    g_prof.stride = every_nth_call;
    return MOE_OK;
}

int moe_profile_calls(void) { return g_prof.calls; }
int moe_profile_stage_count(void) { return ST_COUNT; }
const char* moe_profile_stage_name(int i) { return (i >= 0 && i < ST_COUNT) ? kStageNames[i] : ""; }

int moe_profile_elapsed(int call, float* ms) {
    if (!ms || call < 0 || call >= g_prof.calls) return MOE_ERR_INVALID_ARG;
    for (int i = 0; i < ST_COUNT; ++i) ms[i] = 0.f;
    const size_t base = (size_t)call * kMarks;
    const int m = g_prof.nmarks[call];
    if (m < 2) return MOE_OK;
    if (hipEventSynchronize(g_prof.ev[base + m - 1]) != hipSuccess) return MOE_ERR_HIP;
    for (int i = 1; i < m; ++i) {
        const int st = g_prof.stage[base + i];
        if (st < 0) continue;                  // that event only opened the next stage
        float t = 0.f;
        if (hipEventElapsedTime(&t, g_prof.ev[base + i - 1], g_prof.ev[base + i]) != hipSuccess) return MOE_ERR_HIP;
        ms[st] += t;
    }
    return MOE_OK;
}

}  // extern "C"
