// Gather of the kept tokens fused with the block's first LayerNorm, and the
// plain LayerNorm before the MLP.  One wave per token row; the row is held in
// registers (two-pass mean / biased variance in fp32); 16-byte loads and stores.
// HBM bound: reads k*D bf16, writes k*D bf16.
// The gather launch can also carry the restoration's fill (Sec. 3.3, Eq. 6): the pruned slots of the
// restored map depend only on the selection and on the cached map, not on the block's output, so extra
// workgroups of the same launch write them while the first ones normalise the kept rows.
#include "common.h"
#include "kernels.h"
#include "launch_math.h"
#include "resample.h"

namespace fv {

namespace {

// CH = number of 512-column groups held in registers (D <= 512*CH).
// Row m of the output reads input row (idx ? b*N + idx[m] : m), b = m / k; that
// row index is also written to rows_out[m] when asked for (without idx: the row's token, m % k).
template <int CH>
__device__ __forceinline__ void layernorm_row(const bf16_t* __restrict__ in, const int32_t* __restrict__ idx, int N,
                                              int k, int M, int D, const bf16_t* __restrict__ gamma,
                                              const bf16_t* __restrict__ beta, float eps,
                                              int32_t* __restrict__ rows_out, bf16_t* __restrict__ out, int m) {
    const int lane = threadIdx.x & 63;
    // All kernel arguments are asked for here, together: by itself the compiler fetches them in three dependent rounds
    // behind the branches below, which a launch of few rows cannot hide (eight blocks of 64 rows 533.7 -> 528.3 us).
    asm volatile("" ::"s"(in), "s"(idx), "s"(N), "s"(k), "s"(D), "s"(gamma), "s"(beta), "s"(eps), "s"(rows_out), "s"(out));
    if (m >= M) return;
    size_t src_row = (size_t)m;
    if (idx) src_row = (size_t)(m / k) * N + idx[m];
    if (rows_out && lane == 0) rows_out[m] = idx ? (int32_t)src_row : m % k;
    const bf16_t* src = in + src_row * D;

    // All of the row's loads and the gain / shift loads go out together: one memory
    // latency instead of two in a kernel that has little else to hide it with.
    uint4 raw[CH], graw[CH], braw[CH];
#pragma unroll
    for (int g = 0; g < CH; ++g) {
        const int col = g * 512 + lane * 8;
        if (col < D) {
            raw[g] = *reinterpret_cast<const uint4*>(src + col);
            graw[g] = *reinterpret_cast<const uint4*>(gamma + col);
            braw[g] = *reinterpret_cast<const uint4*>(beta + col);
        }
    }
    layernorm_values<CH>(raw, D, eps, [&](int g) { return graw[g]; }, [&](int g) { return braw[g]; },
                         [&](int g, const uint4& v) {
                             *reinterpret_cast<uint4*>(out + (size_t)m * D + g * 512 + lane * 8) = v;
                         });
}

// The launch's first workgroups clear the counters between them (see ZeroCounters).  Only a call's first LayerNorm
// launch has any; the others run kernels without this (CLEAR; a million rows of 64 columns 229 -> 219 us, four million
// of 8 columns 884 -> 841).
__device__ __forceinline__ void clear_counters(const ZeroCounters& zc) {
    if (!clears_counters(blockIdx.x)) return;
    const CounterShare s = counter_share(blockIdx.x, threadIdx.x, gridDim.x);
    for (int i = s.first; i < zc.n; i += s.step) zc.p[i] = 0;
}

template <int CH, bool CLEAR>
__global__ __launch_bounds__(256) void layernorm_rows_kernel(const bf16_t* __restrict__ in,
                                                             const int32_t* __restrict__ idx, int N, int k,
                                                             int M, int D, const bf16_t* __restrict__ gamma,
                                                             const bf16_t* __restrict__ beta, float eps,
                                                             int32_t* __restrict__ rows_out,
                                                             bf16_t* __restrict__ out, const ZeroCounters zc) {
    if constexpr (CLEAR) clear_counters(zc);
    layernorm_row<CH>(in, idx, N, k, M, D, gamma, beta, eps, rows_out, out, blockIdx.x * 4 + (threadIdx.x >> 6));
}

// The same launch with the restoration's fill behind it: workgroups [0, ln_blocks) normalise the kept rows,
// the others walk the token rows of the restored map (one a wave; to the XCDs in runs or in turn, see xcd_share; ln_blocks
// is a multiple of eight) and write the pruned ones (rank < 0) from the cached map; kept rows are left to the block's last GEMM.
struct FillParams {
    const int32_t* rank;      // [B, N]
    const bf16_t* cache_map;  // [B, hc*wc, D]
    bf16_t* y_out;            // [B, N, D]
    int hc, wc, h, w;
    int shares;   // of a sample, a wave a row
    bool runs;    // in contiguous runs to the XCDs
};
constexpr int kFillRowsPerWave = 1;

template <int CH, bool CLEAR>
__global__ __launch_bounds__(256) void gather_layernorm_fill_kernel(const bf16_t* __restrict__ in,
                                                                    const int32_t* __restrict__ idx, int N, int k,
                                                                    int M, int D, const bf16_t* __restrict__ gamma,
                                                                    const bf16_t* __restrict__ beta, float eps,
                                                                    int32_t* __restrict__ rows_out,
                                                                    bf16_t* __restrict__ out, int ln_blocks,
                                                                    const FillParams f, const ZeroCounters zc) {
    if constexpr (CLEAR) clear_counters(zc);
    if ((int)blockIdx.x < ln_blocks) {
        layernorm_row<CH>(in, idx, N, k, M, D, gamma, beta, eps, rows_out, out, blockIdx.x * 4 + (threadIdx.x >> 6));
        return;
    }
    const int per_sample = xcd_blocks(f.shares, f.runs), fb = blockIdx.x - ln_blocks;
    const int b = fb / per_sample;
    const int blk = xcd_share(fb - b * per_sample, f.shares, f.runs, b);   // (past the end: so are its rows)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int rr = 0; rr < kFillRowsPerWave; ++rr) {
        const int n = (blk * 4 + wave) * kFillRowsPerWave + rr;
        if (n >= N) break;
        if (f.rank[(size_t)b * N + n] >= 0) continue;
        fill_pruned_row_any(f.cache_map + (size_t)b * f.hc * f.wc * D, f.hc, f.wc, f.h, f.w, D, n, lane,
                        f.y_out + ((size_t)b * N + n) * D);
    }
}

// What is left of a product whose K was cut into slices (gemm_sliced.hip): a workgroup adds up the slices of one row, wave w
// the column groups w, w + WAVES, ... of 512, all loads of a group in flight at once, and the residual, and rounds once.  LN: the rows
// meet in LDS and the first wave normalises them, by the LayerNorm launch's own code and from the same rounded values, so a
// row has the bits that two launches would give it.  Bound by the slices' bytes (6.2 TB/s behind 3 us: 960 rows of 2048 columns
// in four slices 8.2 us).
template <int CH, int SPLITS, bool LN>
__global__ __launch_bounds__(64 * (CH < 4 ? CH : 4)) void slice_sum_kernel(const SliceSum p, const bf16_t* __restrict__ gamma,
                                                                          const bf16_t* __restrict__ beta, float eps,
                                                                          bf16_t* __restrict__ a_out) {
    constexpr int WAVES = CH < 4 ? CH : 4;
    __shared__ uint4 row_s[LN ? CH * 64 : 1];
    const int m = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t rrow = p.res_rows ? (size_t)p.res_rows[m] : (size_t)m;
    const size_t orow = p.out_rows ? (size_t)p.out_rows[m] : (size_t)m;
    const size_t slice = (size_t)p.M * p.N;
    uint4 graw[CH], braw[CH];
    if (LN && wave == 0) {
#pragma unroll
        for (int g = 0; g < CH; ++g) {
            const int col = min(g * 512 + lane * 8, p.N - 8);
            graw[g] = *reinterpret_cast<const uint4*>(gamma + col);
            braw[g] = *reinterpret_cast<const uint4*>(beta + col);
        }
    }
#pragma unroll
    for (int g = wave; g < CH; g += WAVES) {
        const int col = g * 512 + lane * 8;
        if (col >= p.N) continue;
        const float* const src = p.slices + (size_t)m * p.N + col;
        f32x4_t v[SPLITS][2];
#pragma unroll
        for (int s = 0; s < SPLITS; ++s)
#pragma unroll
            for (int c = 0; c < 2; ++c) v[s][c] = *reinterpret_cast<const f32x4_t*>(src + s * slice + 4 * c);
        float res[8], o[8];
        unpack8(*reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(p.residual) + rrow * p.N + col), res);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            o[j] = v[0][j >> 2][j & 3];
#pragma unroll
            for (int s = 1; s < SPLITS; ++s) o[j] += v[s][j >> 2][j & 3];
            o[j] += res[j];
        }
        uint4 pk;
        pk.x = pack_bf16x2(o[0], o[1]);
        pk.y = pack_bf16x2(o[2], o[3]);
        pk.z = pack_bf16x2(o[4], o[5]);
        pk.w = pack_bf16x2(o[6], o[7]);
        *reinterpret_cast<uint4*>(static_cast<bf16_t*>(p.out) + orow * p.N + col) = pk;
        if (LN) row_s[g * 64 + lane] = pk;
    }
    if constexpr (LN) {
        __syncthreads();
        if (wave != 0) return;
        uint4 raw[CH];
#pragma unroll
        for (int g = 0; g < CH; ++g) raw[g] = row_s[g * 64 + lane];
        layernorm_values<CH>(raw, p.N, eps, [&](int g) { return graw[g]; }, [&](int g) { return braw[g]; },
                             [&](int g, const uint4& o) {
                                 *reinterpret_cast<uint4*>(a_out + (size_t)m * p.N + g * 512 + lane * 8) = o;
                             });
    }
}

template <int CH, bool LN>
void slice_sum_splits(const SliceSum& s, const bf16_t* gamma, const bf16_t* beta, float eps, bf16_t* a_out, hipStream_t st) {
    const dim3 grid(s.M), block(64 * (CH < 4 ? CH : 4));
    switch (s.splits) {
        case 2: slice_sum_kernel<CH, 2, LN><<<grid, block, 0, st>>>(s, gamma, beta, eps, a_out); break;
        case 4: slice_sum_kernel<CH, 4, LN><<<grid, block, 0, st>>>(s, gamma, beta, eps, a_out); break;
        default: slice_sum_kernel<CH, 8, LN><<<grid, block, 0, st>>>(s, gamma, beta, eps, a_out); break;
    }
}

template <bool LN>
void slice_sum(const SliceSum& s, const void* gamma, const void* beta, float eps, void* a_out, hipStream_t st) {
    const bf16_t* const g = static_cast<const bf16_t*>(gamma);
    const bf16_t* const b = static_cast<const bf16_t*>(beta);
    bf16_t* const a = static_cast<bf16_t*>(a_out);
    const int ch = (s.N + 511) / 512;   // N = D <= 8192
    if (ch <= 1) slice_sum_splits<1, LN>(s, g, b, eps, a, st);
    else if (ch <= 2) slice_sum_splits<2, LN>(s, g, b, eps, a, st);
    else if (ch <= 4) slice_sum_splits<4, LN>(s, g, b, eps, a, st);
    else if (ch <= 8) slice_sum_splits<8, LN>(s, g, b, eps, a, st);
    else slice_sum_splits<16, LN>(s, g, b, eps, a, st);
}

void dispatch(const void* in, const int32_t* idx, int N, int k, int M, int D, const void* gamma,
              const void* beta, float eps, int32_t* rows_out, void* out, const ZeroCounters& zc, hipStream_t stream) {
    const dim3 grid((M + 3) / 4), block(kClearThreads);
    const int ch = (D + 511) / 512;
    const auto launch = [&](auto kernel) {
        kernel<<<grid, block, 0, stream>>>(static_cast<const bf16_t*>(in), idx, N, k, M, D,
                                           static_cast<const bf16_t*>(gamma), static_cast<const bf16_t*>(beta), eps,
                                           rows_out, static_cast<bf16_t*>(out), zc);
    };
#define FV_LN_CASE(CHV) launch(zc.n ? layernorm_rows_kernel<CHV, true> : layernorm_rows_kernel<CHV, false>)
    if (ch <= 1) FV_LN_CASE(1);
    else if (ch <= 2) FV_LN_CASE(2);
    else if (ch <= 4) FV_LN_CASE(4);
    else if (ch <= 8) FV_LN_CASE(8);
    else FV_LN_CASE(16);  // D <= 8192, checked by the caller
#undef FV_LN_CASE
}

}  // namespace

void launch_gather_layernorm(const void* x, const int32_t* idx, int B, int N, int k, int D, const void* gamma,
                             const void* beta, float eps, int32_t* rows_out, void* a_out, const ZeroCounters& zc,
                             hipStream_t stream) {
    dispatch(x, idx, N, k, B * k, D, gamma, beta, eps, rows_out, a_out, zc, stream);
}

void launch_gather_layernorm_fill(const void* x, const int32_t* idx, int B, int N, int k, int D, const void* gamma,
                                  const void* beta, float eps, int32_t* rows_out, void* a_out, const int32_t* rank,
                                  const void* cache_map, int hc, int wc, int h, int w, void* y_out,
                                  const ZeroCounters& zc, hipStream_t stream) {
    const int M = B * k;
    const int ln_blocks = (M + 31) / 32 * 8;
    FillParams f;
    f.rank = rank;
    f.cache_map = static_cast<const bf16_t*>(cache_map);
    f.y_out = static_cast<bf16_t*>(y_out);
    f.hc = hc; f.wc = wc; f.h = h; f.w = w;
    f.shares = (N + 4 * kFillRowsPerWave - 1) / (4 * kFillRowsPerWave);
    f.runs = shares_in_runs(f.shares, w, kFillRowsPerWave);
    const dim3 grid(ln_blocks + B * xcd_blocks(f.shares, f.runs)), block(kClearThreads);
    const int ch = (D + 511) / 512;
    const auto launch = [&](auto kernel) {
        kernel<<<grid, block, 0, stream>>>(static_cast<const bf16_t*>(x), idx, N, k, M, D,
                                           static_cast<const bf16_t*>(gamma), static_cast<const bf16_t*>(beta), eps,
                                           rows_out, static_cast<bf16_t*>(a_out), ln_blocks, f, zc);
    };
#define FV_LNF_CASE(CHV) \
    launch(zc.n ? gather_layernorm_fill_kernel<CHV, true> : gather_layernorm_fill_kernel<CHV, false>)
    if (ch <= 1) FV_LNF_CASE(1);
    else if (ch <= 2) FV_LNF_CASE(2);
    else if (ch <= 4) FV_LNF_CASE(4);
    else if (ch <= 8) FV_LNF_CASE(8);
    else FV_LNF_CASE(16);
#undef FV_LNF_CASE
}

void launch_layernorm(const void* in, int M, int D, const void* gamma, const void* beta, float eps, void* a_out,
                      const ZeroCounters& zc, hipStream_t stream, int32_t* tokens_out, int N) {
    dispatch(in, nullptr, 0, N, M, D, gamma, beta, eps, tokens_out, a_out, zc, stream);
}

void launch_slice_sum(const SliceSum& s, hipStream_t stream) {
    slice_sum<false>(s, nullptr, nullptr, 0.f, nullptr, stream);
}

void launch_slice_sum_layernorm(const SliceSum& s, const void* gamma, const void* beta, float eps, void* a_out,
                                hipStream_t stream) {
    slice_sum<true>(s, gamma, beta, eps, a_out, stream);
}

}  // namespace fv
