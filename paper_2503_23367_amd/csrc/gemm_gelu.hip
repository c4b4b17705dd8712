// The tiled product (gemm_tiles.h) into bias + GELU.
#include "gemm_tiles.h"

namespace fv {

void launch_tiles_gelu(GemmParams& p, hipStream_t stream) { launch_epi<EPI_BIAS_GELU>(p, stream); }

}  // namespace fv
