// Entry of the four-wave tile kernel (ffn_wide.h); an epilogue's instances are compiled in a file of their own.
#include "ffn_wide.h"

namespace moe {

extern template int launch_wide_epi<EPI_STORE>(const WsGemmArgs&, const WsGemmArgs*, int, hipStream_t);
extern template int launch_wide_epi<EPI_GELU>(const WsGemmArgs&, const WsGemmArgs*, int, hipStream_t);
extern template int launch_wide_epi<EPI_SCATTER>(const WsGemmArgs&, const WsGemmArgs*, int, hipStream_t);
extern template int launch_wide_epi<EPI_COMBINE>(const WsGemmArgs&, const WsGemmArgs*, int, hipStream_t);
extern template int launch_wide_epi<EPI_PARTIAL>(const WsGemmArgs&, const WsGemmArgs*, int, hipStream_t);

int launch_wide(const WsGemmArgs& first, const WsGemmArgs* second, int tile_rows, int epi, hipStream_t s) {
    WsGemmArgs a = first, b = second ? *second : first;
    // Groups of at most 128 rows beside one of many: tiles of 256 rows, those of the many first (half-filled tiles cost about
    // 0.7 of a full one here; all on 128-row tiles 157 us, 64 groups x 128 rows + 8192 rows, 4096 x 1024: 150)
    if (second && (a.max_rows > 128) != (b.max_rows > 128)) {
        tile_rows = 256;
        if (b.max_rows > 128) { const WsGemmArgs t = a; a = b; b = t; }
    }
    a.stream = wide_streams(a);
    b.stream = wide_streams(b);
    const WsGemmArgs* pb = second ? &b : nullptr;
    switch (epi) {
        case EPI_STORE: return launch_wide_epi<EPI_STORE>(a, pb, tile_rows, s);
        case EPI_GELU: return launch_wide_epi<EPI_GELU>(a, pb, tile_rows, s);
        case EPI_SCATTER: return second ? MOE_ERR_INVALID_ARG : launch_wide_epi<EPI_SCATTER>(a, pb, tile_rows, s);   // zeroes rows grid-wide
        case EPI_COMBINE: return launch_wide_epi<EPI_COMBINE>(a, pb, tile_rows, s);
        case EPI_PARTIAL: return launch_wide_epi<EPI_PARTIAL>(a, pb, tile_rows, s);
        default: return MOE_ERR_INVALID_ARG;
    }
}

}  // namespace moe
