// The non-expert half of a decoder block for one decode step (one new token per sequence): LayerNorm, attention of
// the new token over its sequence's key/value cache, residual adds.  The paper runs such kernels beside the MoE
// kernels (Sec. 5.4, first paragraph; model shapes in Sec. 3.1) and gives no design for them; everything here is
// bound by memory traffic (the cache is read once per step), so the kernels are plain 16-byte streaming loops.
#include "moe_internal.h"

namespace moe {

__device__ __forceinline__ void unpack8(const uint4 v, float (&f)[8]) {
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    f[4] = __uint_as_float(v.z << 16); f[5] = __uint_as_float(v.z & 0xffff0000u);
    f[6] = __uint_as_float(v.w << 16); f[7] = __uint_as_float(v.w & 0xffff0000u);
}
__device__ __forceinline__ uint4 pack8(const float (&f)[8]) {
    return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
}
// 16 bytes, with the non-temporal hint if they pass through once
template <bool STREAM> __device__ __forceinline__ uint4 load_cache16(const uint16_t* p) {
    if (!STREAM) return *reinterpret_cast<const uint4*>(p);
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)));
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    return v;
}

// A row by one work-group, its pieces of 8 elements held in registers from the sum to the result (NP per thread): one
// memory round trip and the two sums across the waves.  A wave per row with three passes over it, below, left 64 rows to 16
// work-groups: 10.7 us for 64 rows of 2048 with the residual add, 6.6 without.
// SUMS: the added rows are a projection's partial sums, added up here in their order, biased and rounded as the launch that did
// nothing else left them (4.7 us of a step).
template <int NP, bool SUMS>
__global__ __launch_bounds__(256) void add_layernorm_row_kernel(const uint16_t* __restrict__ x, const AddedRows added,
                                                                const float* __restrict__ gamma, const float* __restrict__ beta,
                                                                uint16_t* __restrict__ sum_out, uint16_t* __restrict__ y, int d,
                                                                float eps) {
    __shared__ float part[2][4];
    const uint16_t* r = added.rows;
    const int tid = threadIdx.x, pieces = d / 8;
    const size_t row = (size_t)blockIdx.x * d;
    float f[NP][8], gm[NP][8], bt[NP][8];
    uint4 xv[NP], rv[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {                      // all loads first; past the end: the last piece, not counted
        const int i = min(tid + p * 256, pieces - 1);
        xv[p] = reinterpret_cast<const uint4*>(x + row)[i];
        if constexpr (SUMS) {
            float v[8];
            add_parts8(added.sums, (size_t)gridDim.x * d, row, i, v);
            rv[p] = pack8(v);
        } else if (r) {
            rv[p] = reinterpret_cast<const uint4*>(r + row)[i];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            *reinterpret_cast<float4*>(&gm[p][4 * q]) = reinterpret_cast<const float4*>(gamma)[2 * i + q];
            *reinterpret_cast<float4*>(&bt[p][4 * q]) = reinterpret_cast<const float4*>(beta)[2 * i + q];
        }
    }
    auto block_sum = [&](float v, float (&sh)[4]) {
        v = wave_sum(v);
        if (tid % kWave == 0) sh[tid / kWave] = v;
        __syncthreads();
        return (sh[0] + sh[1]) + (sh[2] + sh[3]);
    };
    float sum = 0.f;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int i = tid + p * 256;
        unpack8(xv[p], f[p]);
        if (SUMS || r) {
            float g[8];
            unpack8(rv[p], g);
#pragma unroll
            for (int q = 0; q < 8; ++q) f[p][q] += g[q];
            const uint4 o = pack8(f[p]);
            unpack8(o, f[p]);                           // the row as it is stored
            if (sum_out && i < pieces) reinterpret_cast<uint4*>(sum_out + row)[i] = o;
        } else if (sum_out && i < pieces) {
            reinterpret_cast<uint4*>(sum_out + row)[i] = xv[p];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) sum += i < pieces ? f[p][q] : 0.f;
    }
    const float mean = block_sum(sum, part[0]) / (float)d;
    float sq = 0.f;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int q = 0; q < 8; ++q) sq += tid + p * 256 < pieces ? (f[p][q] - mean) * (f[p][q] - mean) : 0.f;
    const float rstd = rsqrtf(block_sum(sq, part[1]) / (float)d + eps);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int i = tid + p * 256;
        if (i >= pieces) break;
#pragma unroll
        for (int q = 0; q < 8; ++q) f[p][q] = (f[p][q] - mean) * rstd * gm[p][q] + bt[p][q];
        reinterpret_cast<uint4*>(y + row)[i] = pack8(f[p]);
    }
}

// The same for rows of more than 4096 elements.
// y[t,:] = LayerNorm(s[t,:]) * gamma + beta with s = x (+ r), one wave per row; s is also written to `sum_out` when
// given (rounded to bf16 first: the statistics are those of the stored row).  d is a multiple of 8.
__global__ __launch_bounds__(256) void add_layernorm_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ r,
                                                            const float* __restrict__ gamma, const float* __restrict__ beta,
                                                            uint16_t* __restrict__ sum_out, uint16_t* __restrict__ y, int T,
                                                            int d, float eps) {
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;
    const int pieces = d / 8;
    const uint4* xr = reinterpret_cast<const uint4*>(x + (size_t)t * d);
    const uint4* rr = r ? reinterpret_cast<const uint4*>(r + (size_t)t * d) : nullptr;
    auto row_piece = [&](int i, float (&f)[8]) {
        unpack8(xr[i], f);
        if (rr) {
            float g[8];
            unpack8(rr[i], g);
#pragma unroll
            for (int q = 0; q < 8; ++q) f[q] += g[q];
            unpack8(pack8(f), f);                       // the row as it is stored
        }
    };
    float sum = 0.f;
    for (int i = lane; i < pieces; i += 64) {
        float f[8];
        row_piece(i, f);
        if (sum_out) reinterpret_cast<uint4*>(sum_out + (size_t)t * d)[i] = pack8(f);
#pragma unroll
        for (int q = 0; q < 8; ++q) sum += f[q];
    }
    const float mean = wave_sum(sum) / (float)d;
    float sq = 0.f;
    for (int i = lane; i < pieces; i += 64) {
        float f[8];
        row_piece(i, f);
#pragma unroll
        for (int q = 0; q < 8; ++q) sq += (f[q] - mean) * (f[q] - mean);
    }
    const float rstd = rsqrtf(wave_sum(sq) / (float)d + eps);
    for (int i = lane; i < pieces; i += 64) {
        float f[8];
        row_piece(i, f);
        const float4 g0 = reinterpret_cast<const float4*>(gamma)[2 * i], g1 = reinterpret_cast<const float4*>(gamma)[2 * i + 1];
        const float4 b0 = reinterpret_cast<const float4*>(beta)[2 * i], b1 = reinterpret_cast<const float4*>(beta)[2 * i + 1];
        const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) f[q] = (f[q] - mean) * rstd * g[q] + b[q];
        reinterpret_cast<uint4*>(y + (size_t)t * d)[i] = pack8(f);
    }
}

bool add_layernorm_sums(int d) { return d <= 4096; }
int launch_add_layernorm(const uint16_t* x, const AddedRows& r, const float* gamma, const float* beta, uint16_t* sum_out,
                         uint16_t* y, int T, int d, float eps, hipStream_t s) {
    if (r.sums.partial && (!add_layernorm_sums(d) || r.sums.ksplit < 1 || r.sums.ksplit > kLinearMaxSplit)) return MOE_ERR_INVALID_ARG;
#define MOE_LN_ROW(NP, SUMS) \
    hipLaunchKernelGGL((add_layernorm_row_kernel<NP, SUMS>), dim3(T), dim3(256), 0, s, x, r, gamma, beta, sum_out, y, d, eps)
    if (d <= 2048) {
        if (r.sums.partial) MOE_LN_ROW(1, true);
        else MOE_LN_ROW(1, false);
    } else if (d <= 4096) {
        if (r.sums.partial) MOE_LN_ROW(2, true);
        else MOE_LN_ROW(2, false);
    } else {
        hipLaunchKernelGGL(add_layernorm_kernel, dim3((T + 3) / 4), dim3(256), 0, s, x, r.rows, gamma, beta, sum_out, y, T, d, eps);
    }
#undef MOE_LN_ROW
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// out = a + b, bf16, n8 pieces of 8 elements
__global__ __launch_bounds__(256) void add_rows_kernel(const uint4* __restrict__ a, const uint4* __restrict__ b,
                                                       uint4* __restrict__ out, long long n8) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n8; i += (long long)gridDim.x * 256) {
        float f[8], g[8];
        unpack8(a[i], f);
        unpack8(b[i], g);
#pragma unroll
        for (int q = 0; q < 8; ++q) f[q] += g[q];
        out[i] = pack8(f);
    }
}
int launch_add_rows(const uint16_t* a, const uint16_t* b, uint16_t* out, long long n, hipStream_t s) {
    const long long n8 = n / 8;
    long long blocks = (n8 + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(add_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, s, reinterpret_cast<const uint4*>(a),
                       reinterpret_cast<const uint4*>(b), reinterpret_cast<uint4*>(out), n8);
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

// ---- attention of one new token per sequence over its cache ---------------------------------------------------
// qkv [T, 3d] holds the new token's query, key and value (head h: columns h*DH.. of each third); the caches are
// [T, H, Lmax, DH]; sequence b has pos[b] cached positions and the new token is position pos[b].
// A work-group takes kAttnChunk consecutive positions of one (sequence, head); LPP = DH/8 lanes share a position
// (16 bytes of its key and value each), a wave step covers 64/LPP consecutive positions = 1 KB of contiguous cache.
// Every lane group keeps a running softmax (maximum, sum, weighted values); the groups of a work-group meet in LDS
// and leave one partial (m, l, o[DH]) per chunk.
// attn_merge_kernel merges them; a sequence's only chunk is the result, and with room for one chunk there is no merge.
// (Merged by the work-group of a sequence and head that comes last, every work-group pays for the hand-over across the XCDs' L2s:
// 64 sequences of 16 heads, 8 chunks 92.9 + 4.6 -> 99.8 us; 107 of 8, 4 chunks 35 + 4.8 -> 46.6; 10 of 8, 3 chunks 8.1 + 3.9 -> 11.2.)
// The chunk that holds position pos[b]
// takes the new key/value from qkv, never from the cache, so the write of the new rows into the cache (by chunk 0)
// races with nobody.
// Bound by the read of the cache: kAttnAhead steps are loaded together and meet in one rescaling of the running softmax
// (one step at a time, load after use, ran at 5 TB/s: 108 us for 64 sequences of 2048 positions at most, 16 heads of 128).
constexpr int kAttnChunk = 256;
constexpr int kAttnAhead = 4;

// cached positions (clamped into the cache: no access can leave it), and chunks with a position: the new token is position npast
__device__ __forceinline__ int past_positions(int pos, int Lmax) { return min(max(pos, 0), Lmax - 1); }
__device__ __forceinline__ int live_chunks(int pos, int Lmax) { return past_positions(pos, Lmax) / kAttnChunk + 1; }

// Element t of a (sequence, head)'s result from its chunks' partials
template <int DH> __device__ __forceinline__ uint16_t merge_chunks(const float* p, int nlive, int t) {
    // sum_split o exp(m - M) / sum_split l exp(m - M), eight chunks' partials in flight; a chunk whose scores are all NaN holds
    // m = -inf and NaN
    float M = -INFINITY, L = 0.f, O = 0.f;
    for (int s0 = 0; s0 < nlive; s0 += 8) {
        float mu[8], lu[8], ou[8], mn = M;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float* ps = p + min(s0 + u, nlive - 1) * (DH + 2);
            mu[u] = s0 + u < nlive ? ps[0] : -INFINITY;
            lu[u] = s0 + u < nlive ? ps[1] : 0.f;
            ou[u] = s0 + u < nlive ? ps[2 + t] : 0.f;              // not the last chunk's once more: 0 times infinity is NaN
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) mn = fmaxf(mn, mu[u]);
        const float c = M == mn ? 1.f : __expf(M - mn);
        L *= c;
        O *= c;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float e = s0 + u >= nlive ? 0.f : mu[u] == mn ? 1.f : __expf(mu[u] - mn);
            L = fmaf(lu[u], e, L);
            O = fmaf(ou[u], e, O);
        }
        M = mn;
    }
    return f32_to_bf16(O / L);
}

template <int DH, bool STREAM>
__global__ __launch_bounds__(256) void attn_decode_kernel(const uint16_t* __restrict__ qkv, uint16_t* __restrict__ cache_k,
                                                          uint16_t* __restrict__ cache_v, const int32_t* __restrict__ pos,
                                                          float* __restrict__ partial, uint16_t* __restrict__ attn,
                                                          int H, int Lmax, int nsplit) {
    constexpr int LPP = DH / 8, PPW = 64 / LPP, NG = 4 * PPW;       // lanes per position, positions per wave step, groups
    __shared__ float m_sh[NG], l_sh[NG];
    __shared__ float o_sh[NG][DH];
    const int bh = blockIdx.x, b = bh / H, h = bh % H, split = blockIdx.y;
    const int d = H * DH;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int sub = lane % LPP, grp = lane / LPP;
    const int npast = past_positions(pos[b], Lmax);
    const int nlive = live_chunks(npast, Lmax);
    if (split >= nlive) return;
    const uint16_t* qrow = qkv + (size_t)b * 3 * d + h * DH;
    float q[8];
    unpack8(*reinterpret_cast<const uint4*>(qrow + sub * 8), q);
    const float scale = rsqrtf((float)DH);
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] *= scale;
    const uint16_t* kc = cache_k + ((size_t)b * H + h) * Lmax * DH;
    const uint16_t* vc = cache_v + ((size_t)b * H + h) * Lmax * DH;
    if (split == 0 && tid < 2 * LPP) {                               // the new rows join the cache for later steps
        const int which = tid / LPP, piece = tid % LPP;
        const uint4 v = *reinterpret_cast<const uint4*>(qrow + (1 + which) * d + piece * 8);
        uint16_t* dst = (which ? cache_v : cache_k) + (((size_t)b * H + h) * Lmax + npast) * DH + piece * 8;
        *reinterpret_cast<uint4*>(dst) = v;
    }
    float m = -INFINITY, l = 0.f, o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = 0.f;
    const int p0 = split * kAttnChunk + w * (kAttnChunk / 4);
    const uint4 knew = *reinterpret_cast<const uint4*>(qrow + d + sub * 8);       // the new token itself
    const uint4 vnew = *reinterpret_cast<const uint4*>(qrow + 2 * d + sub * 8);
    static_assert(kAttnChunk / 4 / PPW % kAttnAhead == 0, "whole rounds");
    for (int step = 0; step < kAttnChunk / 4 / PPW; step += kAttnAhead) {
        if (p0 + step * PPW > npast) break;                          // uniform over the wave
        uint4 kraw[kAttnAhead], vraw[kAttnAhead];
#pragma unroll
        for (int u = 0; u < kAttnAhead; ++u) {
            const int pc = min(p0 + (step + u) * PPW + grp, max(npast - 1, 0));   // clamped cache position (in bounds; unused past npast)
            kraw[u] = load_cache16<STREAM>(kc + (size_t)pc * DH + sub * 8);
            vraw[u] = load_cache16<STREAM>(vc + (size_t)pc * DH + sub * 8);
        }
        float s[kAttnAhead], mn = m;
        bool some = false;
#pragma unroll
        for (int u = 0; u < kAttnAhead; ++u) {
            const int p = p0 + (step + u) * PPW + grp;
            float kf[8];
            unpack8(p == npast ? knew : kraw[u], kf);
            s[u] = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) s[u] = fmaf(q[i], kf[i], s[u]);
#pragma unroll
            for (int msk = 1; msk < LPP; msk <<= 1) s[u] += __shfl_xor(s[u], msk);
            if (p > npast) s[u] = -INFINITY;
            some = some || !(s[u] == -INFINITY);                     // NaN is a score: it has to reach l (fmaxf passes it over)
            mn = fmaxf(mn, s[u]);
        }
        if (some) {                                                  // false: no position for this lane group
            const float c = __expf(m - mn);                          // m = -inf at first: c = 0
            l *= c;
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] *= c;
#pragma unroll
            for (int u = 0; u < kAttnAhead; ++u) {
                const float e = __expf(s[u] - mn);                   // exp(-inf) = 0 past npast
                float vf[8];
                const int p = p0 + (step + u) * PPW + grp;
                unpack8(p < npast ? vraw[u] : p == npast ? vnew : make_uint4(0, 0, 0, 0), vf);   // past npast: 0 times 0
                l += e;
#pragma unroll
                for (int i = 0; i < 8; ++i) o[i] = fmaf(e, vf[i], o[i]);
            }
            m = mn;
        }
    }
    const int g = w * PPW + grp;
    if (sub == 0) { m_sh[g] = m; l_sh[g] = l; }
#pragma unroll
    for (int i = 0; i < 8; ++i) o_sh[g][sub * 8 + i] = o[i];
    __syncthreads();
    if (tid < DH) {
        float M = -INFINITY;
        for (int j = 0; j < NG; ++j) M = fmaxf(M, m_sh[j]);
        float L = 0.f, O = 0.f;
        for (int j = 0; j < NG; ++j) {
            // empty groups: exp(-inf) = 0; M = -inf: nothing but empty groups and such whose scores were all NaN (l is NaN)
            const float c = m_sh[j] == M ? 1.f : __expf(m_sh[j] - M);
            L = fmaf(l_sh[j], c, L);
            O = fmaf(o_sh[j][tid], c, O);
        }
        if (nlive == 1) {
            attn[(size_t)bh * DH + tid] = f32_to_bf16(O / L);
        } else {
            float* dst = partial + ((size_t)bh * nsplit + split) * (DH + 2);
            dst[2 + tid] = O;
            if (tid == 0) { dst[0] = M; dst[1] = L; }
        }
    }
}

template <int DH>
__global__ __launch_bounds__(DH) void attn_merge_kernel(const float* __restrict__ partial, const int32_t* __restrict__ pos, uint16_t* __restrict__ attn,
                                                        int H, int Lmax, int nsplit) {
    const int bh = blockIdx.x, nlive = live_chunks(pos[bh / H], Lmax);
    if (nlive > 1) attn[(size_t)bh * DH + threadIdx.x] = merge_chunks<DH>(partial + (size_t)bh * nsplit * (DH + 2), nlive, threadIdx.x);
}

int attn_nsplit(int Lmax) { return (Lmax + kAttnChunk - 1) / kAttnChunk; }
size_t attn_partial_floats(int T, int H, int dh, int Lmax) { return (size_t)T * H * attn_nsplit(Lmax) * (dh + 2); }
bool attn_supported(int d, int H) { return H >= 1 && d % H == 0 && (d / H == 64 || d / H == 128); }

int launch_attn_decode(const uint16_t* qkv, uint16_t* cache_k, uint16_t* cache_v, const int32_t* pos, float* partial,
                       uint16_t* attn, int T, int H, int dh, int Lmax, hipStream_t s) {
    const int nsplit = attn_nsplit(Lmax);
    const dim3 grid((unsigned)(T * H), (unsigned)nsplit);
    // Caches beyond the 256 MB Infinity Cache stream past it (blocks of 64 sequences, d = 2048, 2048 positions: 705 -> 687 us;
    // 128, d = 1024, 1500: 216 -> 206); smaller ones are read from there at the next step (32, d = 1024, 2000: 132 -> 134).  The rule
    // sees the room for positions only: short sequences in a large cache pay for the hint (up to 256 of 2048 positions, block
    // without much of a feed-forward part: 108.6 -> 112.5; all 2048: 202 -> 184).
    const bool stream = (long long)T * H * Lmax * dh * 4 > 256ll << 20;
#define MOE_ATTN(DH, STREAM) \
    hipLaunchKernelGGL((attn_decode_kernel<DH, STREAM>), grid, dim3(256), 0, s, qkv, cache_k, cache_v, pos, partial, attn, H, Lmax, nsplit)
#define MOE_ATTN_MERGE(DH) \
    if (nsplit > 1) hipLaunchKernelGGL((attn_merge_kernel<DH>), dim3((unsigned)(T * H)), dim3(DH), 0, s, partial, pos, attn, H, Lmax, nsplit)
    if (dh == 128) {
        if (stream) MOE_ATTN(128, true);
        else MOE_ATTN(128, false);
        MOE_ATTN_MERGE(128);
    } else {
        if (stream) MOE_ATTN(64, true);
        else MOE_ATTN(64, false);
        MOE_ATTN_MERGE(64);
    }
#undef MOE_ATTN_MERGE
#undef MOE_ATTN
    return hipGetLastError() == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

}  // namespace moe
