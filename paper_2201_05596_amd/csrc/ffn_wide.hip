// Entry of the four-wave tile kernel (ffn_wide.h); an epilogue's instances are compiled in a file of their own.
#include "ffn_wide.h"

namespace moe {

extern template int launch_wide_epi<EPI_STORE>(const WsGemmArgs&, const WsGemmArgs*, int, int, hipStream_t);
extern template int launch_wide_epi<EPI_GELU>(const WsGemmArgs&, const WsGemmArgs*, int, int, hipStream_t);
extern template int launch_wide_epi<EPI_SCATTER>(const WsGemmArgs&, const WsGemmArgs*, int, int, hipStream_t);
extern template int launch_wide_epi<EPI_PARTIAL>(const WsGemmArgs&, const WsGemmArgs*, int, int, hipStream_t);

// Both halves of an FFN have weights of this size: beyond 128 MB a pass evicts what the next one would have found in the
// Infinity Cache.  (64 groups x 128 rows x 4096 x 1024, 537 MB: 105 -> 91 us with the hint, 16 rows 89 -> 79 = 6.8 TB/s; 32
// groups x 16 rows, 268 MB read again and again 41 -> 48; weights that several row tiles read, 8192 x 4096 x 4096 193 -> 212.)
static bool wide_streams(const WsGemmArgs& a) { return (long long)a.G * a.K * a.N * 2 > (128ll << 20); }

int wide_policy(const WsGemmArgs& a, const WsGemmArgs* b, int tile_rows, int epi) {
    if (!wide_hints(epi)) return WIDE_CACHED;
    const bool sa = wide_streams(a), sb = b && wide_streams(*b);
    if (sa && a.max_rows <= tile_rows && (!b || (sb && b->max_rows <= tile_rows))) return WIDE_STREAMED;
    return tile_rows == 256 && (sa || sb) ? WIDE_BY_GROUP : WIDE_CACHED;
}

int launch_wide(const WsGemmArgs& first, const WsGemmArgs* second, int tile_rows, int epi, hipStream_t s) {
    WsGemmArgs a = first, b = second ? *second : first;
    if (second && b.max_rows > 128 && a.max_rows <= 128) { const WsGemmArgs t = a; a = b; b = t; }   // the full tiles first
    a.stream = wide_streams(a);
    b.stream = wide_streams(b);
    const WsGemmArgs* pb = second ? &b : nullptr;
    const int policy = wide_policy(a, pb, tile_rows, epi);
    switch (epi) {
        case EPI_STORE: return launch_wide_epi<EPI_STORE>(a, pb, tile_rows, policy, s);
        case EPI_GELU: return launch_wide_epi<EPI_GELU>(a, pb, tile_rows, policy, s);
        case EPI_SCATTER: return second ? MOE_ERR_INVALID_ARG : launch_wide_epi<EPI_SCATTER>(a, pb, tile_rows, policy, s);   // zeroes rows grid-wide
        case EPI_PARTIAL: return launch_wide_epi<EPI_PARTIAL>(a, pb, tile_rows, policy, s);
        default: return MOE_ERR_INVALID_ARG;
    }
}

}  // namespace moe
