// Instances of the four-wave tile kernel (ffn_wide.h).
#include "ffn_wide.h"

namespace moe {

template int launch_wide_epi<EPI_SCATTER>(const WsGemmArgs&, const WsGemmArgs*, int, int, hipStream_t);

}  // namespace moe
