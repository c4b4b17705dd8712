// Where a product goes: few rows, slices of K, or whole tiles.
#include "gemm_tiles.h"

namespace fv {

SplitKPlan residual_product_plan(int M, int N, int K, SlicesMeet meet) {
    return gemm_cfg_override(EPI_BIAS_RES) >= 0 ? SplitKPlan{} : gemm_splitk_plan(M, N, K, meet);
}

void launch_gemm(GemmEpilogue epi, const GemmArgs& a, hipStream_t stream) {
    if (few_rows_product(a.M, a.N, a.K, a.slice_ws && few_rows_tiled_splits(a.N, a.K))) {
        launch_gemm_skinny(epi, a, stream);
        return;
    }
    GemmParams p;
    p.A = static_cast<const bf16_t*>(a.A);
    p.W = static_cast<const bf16_t*>(a.W);
    p.bias = static_cast<const bf16_t*>(a.bias);
    p.M = a.M; p.N = a.N; p.K = a.K;
    p.out = static_cast<bf16_t*>(a.out);
    p.residual = static_cast<const bf16_t*>(a.residual);
    p.res_rows = a.res_rows;
    p.out_rows = a.out_rows;
    p.q_out = static_cast<bf16_t*>(a.q_out);
    p.k_cache = static_cast<bf16_t*>(a.k_cache);
    p.v_cache = static_cast<bf16_t*>(a.v_cache);
    p.D = a.D; p.H = a.H; p.dh = a.dh; p.k_tokens = a.k_tokens; p.L0 = a.L0; p.L_cap = a.L_cap;
    p.rope_cos = a.rope_cos; p.rope_sin = a.rope_sin; p.rope_rows = a.rope_rows; p.rope_N = a.rope_N;
    p.tiles_m = p.tiles_n = 0;
    p.splits = 1;
    p.slices = static_cast<float*>(a.slice_ws);
    if (epi == EPI_BIAS_RES && a.slices.splits > 1) {
        launch_tiles_sliced(a.slices, p, stream);
        return;
    }
    switch (epi) {
        case EPI_QKV:
            if (a.rope_cos) launch_tiles_rope(p, stream);
            else launch_tiles_qkv(p, stream);
            break;
        case EPI_BIAS_RES: launch_tiles_residual(p, stream); break;
        case EPI_BIAS_GELU: launch_tiles_gelu(p, stream); break;
    }
}

}  // namespace fv
