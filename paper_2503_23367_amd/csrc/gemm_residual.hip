// The tiled product (gemm_tiles.h) into bias + residual.
#include "gemm_tiles.h"

namespace fv {

void launch_tiles_residual(GemmParams& p, hipStream_t stream) { launch_epi<EPI_BIAS_RES>(p, stream); }

}  // namespace fv
