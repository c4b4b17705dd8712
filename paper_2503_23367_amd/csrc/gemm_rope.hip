// The tiled product (gemm_tiles.h) into the query buffer and the KV caches, with rotary positions.
#include "gemm_tiles.h"

namespace fv {

void launch_tiles_rope(GemmParams& p, hipStream_t stream) { launch_epi<EPI_QKV_ROPE>(p, stream); }

}  // namespace fv
