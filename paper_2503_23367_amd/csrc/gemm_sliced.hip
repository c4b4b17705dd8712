// The tiled product (gemm_tiles.h) with its K range cut into slices.
#include "gemm_tiles.h"

namespace fv {

void launch_tiles_sliced(const SplitKPlan& sk, GemmParams& p, hipStream_t stream) {
    p.splits = sk.splits;
    switch (sk.cfg) {
        case TILE_64x64: launch_cfg<64, 64, 64, 8, 2, 2, 1, EPI_BIAS_RES, true>(p, stream); break;
        case TILE_128x64: launch_cfg<128, 64, 64, 6, 4, 2, 1, EPI_BIAS_RES, true>(p, stream); break;
        case TILE_192x128: launch_cfg<192, 128, 64, 3, 2, 4, 1, EPI_BIAS_RES, true>(p, stream); break;
        case TILE_160x128: launch_cfg<160, 128, 64, 4, 2, 2, 1, EPI_BIAS_RES, true>(p, stream); break;
        default: launch_cfg<128, 128, 64, 4, 2, 4, 1, EPI_BIAS_RES, true>(p, stream); break;   // TILE_128x128
    }
}

}  // namespace fv
