// The tiled product (gemm_tiles.h) into the query buffer and the KV caches.
#include "gemm_tiles.h"

namespace fv {

void launch_tiles_qkv(GemmParams& p, hipStream_t stream) { launch_epi<EPI_QKV>(p, stream); }

}  // namespace fv
