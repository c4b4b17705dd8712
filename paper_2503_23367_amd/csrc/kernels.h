// Host-side launchers of the gfx950 kernels (internal to the library).
// Every launcher enqueues on `stream` and returns; shapes are validated by the
// C-ABI layer before any launcher is called.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>

#include "launch_math.h"
#include "prefetch.h"

namespace fv {

// Raises a kernel's dynamic-LDS limit: a per-function attribute that has to be set once per process before
// the first launch that asks for more than 64 KB.  The once_flag (one per launch site, i.e. per kernel
// instantiation) makes concurrent first calls from several host threads safe.
template <class Kernel>
inline void raise_lds_limit_once(std::once_flag& once, Kernel kernel, size_t bytes) {
    std::call_once(once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)bytes);
    });
}

// ---- selection (Sec. 3.3, Eq. 4-5) ----
struct SelectPlan {
    int n_chunks;        // row chunks of the column-sum pass
    int rows_per_chunk;
    size_t off_partial;  // fp64 [B, n_chunks, D]
    size_t off_score;    // fp32 [B, N]
    size_t bytes;
};
SelectPlan select_plan(int B, int N, int D);
// idx [B, k] and rank [B, N] (optional); with k == 0 or k == N the result does not depend on x and only
// score_out, if asked for, is computed from it.
void launch_select(const void* x, int B, int N, int D, int k, int32_t* idx, int32_t* rank,
                   float* score_out, void* ws, const SelectPlan& plan, hipStream_t stream);
// The index list of a selection that keeps every token.
void launch_keep_all(int32_t* idx, int B, int N, hipStream_t stream);

// ---- restoration (Sec. 3.3, Eq. 6) ----
void launch_rank_from_idx(const int32_t* idx, int32_t* rank, int B, int N, int k, hipStream_t stream);
void launch_restore(const void* y_kept, const int32_t* rank, int B, int k, const void* cache_map,
                    int hc, int wc, int h, int w, int D, void* y_out, hipStream_t stream);
// Eq. 2 on fp32 maps [B, h*w, C] (C % 4 == 0): r_out = resample(r_prev [B, hp*wp, C]) + f_k (bf16).
// r_prev or f_k may be null (not both).
void launch_residual_accumulate(const float* r_prev, int hp, int wp, const void* f_k, int h, int w, int B, int C,
                                float* r_out, hipStream_t stream);

// ---- block pieces ----
// Arrival counters in the caller's scratch that have to be zero before the call's first attention launch
// (its key ranges; every kernel that uses them leaves them zero again).  The call's first LayerNorm launch
// clears them on the side, which costs nothing measurable; a launch of their own cost 2.7 us.
struct ZeroCounters {
    int32_t* p = nullptr;
    int n = 0;
};
// xk = x[idx] (optional copy out) and a = LayerNorm(xk); one wave per row.
// rows_out (optional, int32 [B*k]) receives the absolute source row b*N + idx[m] of
// every kept token, for later gathers of the same rows.
void launch_gather_layernorm(const void* x, const int32_t* idx, int B, int N, int k, int D,
                             const void* gamma, const void* beta, float eps, int32_t* rows_out,
                             void* a_out, const ZeroCounters& zc, hipStream_t stream);
// The same launch carrying the restoration's fill as well (Sec. 3.3, Eq. 6): extra workgroups write every
// pruned row (rank[b,n] < 0) of y_out [B, N, D] from cache_map [B, hc*wc, D] resampled to h x w (N = h*w).
// y_out must not be x.  Kept rows of y_out are not touched.
void launch_gather_layernorm_fill(const void* x, const int32_t* idx, int B, int N, int k, int D, const void* gamma,
                                  const void* beta, float eps, int32_t* rows_out, void* a_out, const int32_t* rank,
                                  const void* cache_map, int hc, int wc, int h, int w, void* y_out,
                                  const ZeroCounters& zc, hipStream_t stream);
// a = LayerNorm(rows of `in`), M rows.  tokens_out [M] (optional): every row's token, m % N.
void launch_layernorm(const void* in, int M, int D, const void* gamma, const void* beta, float eps,
                      void* a_out, const ZeroCounters& zc, hipStream_t stream, int32_t* tokens_out = nullptr, int N = 1);

enum GemmEpilogue {
    EPI_QKV = 0,       // +bias; q -> q_out [M, D]; k, v -> caches at positions L0 + t
    EPI_BIAS_RES = 1,  // out = acc + bias + residual
    EPI_BIAS_GELU = 2  // out = gelu(acc + bias)
};
// Internal fourth epilogue: EPI_QKV with the rotary embedding of q and the new keys (an instantiation of its
// own, so that the plain QKV GEMM carries none of its registers).
constexpr int EPI_QKV_ROPE = 3;
constexpr bool is_qkv(int epi) { return epi == EPI_QKV || epi == EPI_QKV_ROPE; }
struct GemmArgs {
    const void* A;     // [M, K] bf16
    const void* W;     // [N, K] bf16
    const void* bias;  // [N] bf16 or null
    int M, N, K;
    // EPI_BIAS_RES / EPI_BIAS_GELU
    void* out;             // [M, N] bf16
    const void* residual;  // [M, N] bf16 (EPI_BIAS_RES), or the gather source when res_idx is set
    const int32_t* res_rows = nullptr;  // optional: the residual of output row m is row res_rows[m] of `residual`
    const int32_t* out_rows = nullptr;  // optional (EPI_BIAS_RES): output row m is written to row out_rows[m] of `out`
    // EPI_QKV
    void* q_out;    // [M, D]
    void* k_cache;  // [B, H, L_cap, dh]
    void* v_cache;  // [B, H, dh, L_cap]
    int D, H, dh, k_tokens, L0, L_cap;
    // EPI_QKV, optional: rotary embedding of q and the new keys.  rope_cos / rope_sin [rope_N, dh/2] fp32
    // (launch_rope2d_table); the slot of output row m is rope_rows[m] % rope_N (a row list that is absolute,
    // b*N + n, or per sample, n, gives the same slot), or with rope_rows == NULL its token index m % k_tokens.
    const float* rope_cos = nullptr;
    const float* rope_sin = nullptr;
    const int32_t* rope_rows = nullptr;
    int rope_N = 0;
    // Optional scratch of a block's products, and how K is cut (EPI_BIAS_RES; residual_product_plan, which also says how much of the
    // scratch it takes).  Cut, the launch leaves its slices there and touches neither `out` nor `residual`: the launch of a
    // SliceSum has to follow.
    void* slice_ws = nullptr;
    SplitKPlan slices;
    // Optional (EPI_QKV, EPI_BIAS_GELU; only where few_rows_layernorm says so): the rows of A are normalised on
    // the way in, and the call's arrival counters cleared, as the LayerNorm launch this replaces would.
    const void* ln_g = nullptr;
    const void* ln_b = nullptr;
    float ln_eps = 0.f;
    ZeroCounters zero;
};
void launch_gemm(GemmEpilogue epi, const GemmArgs& a, hipStream_t stream);

// GEMMs of few rows (skinny.hip); launch_gemm routes there what few_rows_product (launch_math.h) gives it.
void launch_gemm_skinny(GemmEpilogue epi, const GemmArgs& a, hipStream_t stream);

// The plan of an out-proj or FC2 product (EPI_BIAS_RES) for GemmArgs: gemm_splitk_plan, and no slices where a tuning build forces
// a tile.
SplitKPlan residual_product_plan(int M, int N, int K, SlicesMeet meet);
// What is left of a split product: out[row] = sum of the slices, in slice order, + residual (the bias is in the first slice).
struct SliceSum {
    const float* slices = nullptr;   // [splits][M][N]; null: nothing is left to do
    int splits = 0, M = 0, N = 0;
    const void* residual = nullptr;
    const int32_t* res_rows = nullptr;   // as in GemmArgs
    const int32_t* out_rows = nullptr;
    void* out = nullptr;
};
// The sum alone, or with the LayerNorm of the rows behind it: a_out[m] = LayerNorm(out row of m).
void launch_slice_sum(const SliceSum& s, hipStream_t stream);
void launch_slice_sum_layernorm(const SliceSum& s, const void* gamma, const void* beta, float eps, void* a_out,
                                hipStream_t stream);
// cos / sin tables [h*w, dh/2] fp32 of the axial 2-D rotary embedding (see rope.hip).
void launch_rope2d_table(int h, int w, int dh, double base, int ref_h, int ref_w, float* cos_out, float* sin_out,
                         hipStream_t stream);

// Matrices that the products behind a launch read, in that order.
struct WeightsAhead {
    const void* p[Prefetch::kRanges] = {};
    long bytes[Prefetch::kRanges] = {};
    int n = 0;
    void add(const void* w, long size) { p[n] = w; bytes[n++] = size; }
    // What a launch of `us` microseconds with `idle` idle CUs fetches of them (prefetch_plan).
    Prefetch plan(int idle, double us, bool cut) const {
        Prefetch f;
        PrefetchPlan pl = prefetch_plan(bytes, n, idle, us, cut);
        f.blocks = pl.blocks;
        for (int i = 0; i < n && pl.bytes >= 128; ++i) {
            const long take = bytes[i] < pl.bytes ? bytes[i] : pl.bytes;
            f.p[i] = static_cast<const char*>(p[i]);
            f.lines[i] = (int)(take / 128);
            pl.bytes -= take;
        }
        return f;
    }
};

struct AttnArgs {
    const void* q;        // [B*k, D] bf16 (feature = head*dh + d)
    const void* k_cache;  // [B, H, L_cap, dh]
    const void* v_cache;  // [B, H, dh, L_cap]
    void* o;              // [B*k, D] bf16
    int B, H, dh, k_tokens, L, L_cap;
    float scale;
    // Optional scratch (attention_split_plan) that lets shapes with too few queries to fill the chip
    // split the key range between workgroups; without it every workgroup walks all keys.
    void* split_ws = nullptr;
    size_t split_ws_bytes = 0;   // its size: variants that need more are not considered
    WeightsAhead ahead;          // fetched by a launch that leaves CUs idle
};
void launch_attention(const AttnArgs& a, hipStream_t stream);

// Key-range split for attention shapes whose workgroups do not fill whole rounds of 256 CUs (too few
// queries, or a last round that is mostly empty): `splits` workgroups per query tile each take
// `keys_per_split` keys (a multiple of the key tile) and leave unnormalised partial outputs with their
// softmax statistics in scratch; the workgroup that finishes a query tile last merges them (softmax
// partials combine exactly; it adds them in range order, so the result does not depend on who was last).
// The plan is the cheapest of 128- or 256-query workgroups on 2-4 key ranges, for every tile or only for
// the tiles of a part-filled last round (the whole rounds before it stay unsplit), under a simple
// round-count model, if that beats the unsplit launch.  splits == 1: no scratch.  max_bytes != 0: only variants whose
// scratch fits.
struct AttnSplitPlan {
    int splits;
    int keys_per_split;
    bool wide;      // 256-query workgroups (else 128-query ones)
    int full_tiles;        // (sample, head, query tile) triples walked whole by one workgroup (whole rounds of 256)
    int tail_tiles;        // the others, shared by `splits` workgroups each
    int counters;          // arrival counters at the head of the scratch (zero on entry, zero again on exit)
    size_t counter_bytes;
    size_t bytes;          // counters + partial results
};
AttnSplitPlan attention_split_plan(int B, int H, int dh, int k_tokens, int L, size_t max_bytes = 0);

}  // namespace fv
