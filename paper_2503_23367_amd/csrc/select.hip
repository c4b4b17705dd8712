// Pivotal Token Selection (FastVAR Sec. 3.3, Eq. 4-5): per-channel mean over
// the token positions, squared distance of every token from it, and the k
// highest-scoring tokens per sample.
//
// Three launches, all bit-reproducible (no floating-point atomics):
//   colsum   fp64 column sums of a few long row chunks            (HBM bound: reads x once)
//   score    every workgroup adds the chunk sums to the mean by itself (a few
//            chunks only, so that this stays cheap), then fp64
//            sum_c (x - mean)^2 per token, rounded once to fp32    (re-reads x, mostly from cache)
//   topk     one workgroup per sample: equal-width bins over the range of the scores'
//            order-preserving bit patterns, direct ranking inside the bin that the
//            k-th falls into, then an ordered compaction (ties to the lowest index)
// A selection that keeps every token or none does not depend on the scores: one fill launch.
#include "common.h"
#include "kernels.h"
#include "launch_math.h"

namespace fv {

namespace {

__device__ __forceinline__ void add8(double (&acc)[8], const uint4& v) {
    acc[0] += (double)bf16_lo(v.x);
    acc[1] += (double)bf16_hi(v.x);
    acc[2] += (double)bf16_lo(v.y);
    acc[3] += (double)bf16_hi(v.y);
    acc[4] += (double)bf16_lo(v.z);
    acc[5] += (double)bf16_hi(v.z);
    acc[6] += (double)bf16_lo(v.w);
    acc[7] += (double)bf16_hi(v.w);
}

// grid (ceil(D/64), n_chunks, B), block 256: column sums of the row chunk for 64 columns (eight lanes read the
// 128 bytes of a row, 32 rows per pass, eight passes of loads in flight), combined through LDS in a fixed order.
// Few, long chunks: the launch after this one sums them in every workgroup, which it can only do cheaply for a
// handful (4096 x 2048: 8 chunks, 128 KB of partials), and that takes a launch of its own (4.7 us) off the
// selection, for 1.5 us more in the score launch; 256 workgroups with 32 KB in flight each read x about as fast as more and
// shorter ones (5.5 against 5.2 us).  The selection inside the step of 4096 x 2048: 27.5 -> 21.2 us in all.
constexpr int kColRows = 32;      // rows of a pass
__global__ __launch_bounds__(256) void colsum_kernel(const bf16_t* __restrict__ x, double* __restrict__ partial, int N,
                                                     int D, int rows_per_chunk, int n_chunks) {
    __shared__ double red[kColRows][kColTile];
    __shared__ double red4[4][kColTile];
    const int c8 = threadIdx.x & 7, rr = threadIdx.x >> 3;
    const int col = blockIdx.x * kColTile + c8 * 8;
    const int b = blockIdx.z;
    const int r0 = blockIdx.y * rows_per_chunk;
    const int r1 = min(r0 + rows_per_chunk, N);

    double acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.0;
    if (col < D) {
        const bf16_t* base = x + (size_t)b * N * D + col;
        int r = r0 + rr;
        for (; r + 7 * kColRows < r1; r += 8 * kColRows) {
            uint4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const uint4*>(base + (size_t)(r + u * kColRows) * D);
#pragma unroll
            for (int u = 0; u < 8; ++u) add8(acc, v[u]);
        }
        for (; r < r1; r += kColRows) {
            const uint4 v0 = *reinterpret_cast<const uint4*>(base + (size_t)r * D);
            add8(acc, v0);
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[rr][c8 * 8 + j] = acc[j];
    __syncthreads();
    const int cl = threadIdx.x & 63, g = threadIdx.x >> 6;
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < kColRows / 4; ++j) s += red[g * (kColRows / 4) + j][cl];
    red4[g][cl] = s;
    __syncthreads();
    if (g == 0) {
        const int c = blockIdx.x * kColTile + cl;
        if (c < D)
            partial[((size_t)b * n_chunks + blockIdx.y) * D + c] =
                ((red4[0][cl] + red4[1][cl]) + red4[2][cl]) + red4[3][cl];
    }
}

__device__ __forceinline__ void sqdev8(double& acc, const uint4& v, const double* mu /* stride 64 */) {
    double d;
    d = (double)bf16_lo(v.x) - mu[0 * 64]; acc = fma(d, d, acc);
    d = (double)bf16_hi(v.x) - mu[1 * 64]; acc = fma(d, d, acc);
    d = (double)bf16_lo(v.y) - mu[2 * 64]; acc = fma(d, d, acc);
    d = (double)bf16_hi(v.y) - mu[3 * 64]; acc = fma(d, d, acc);
    d = (double)bf16_lo(v.z) - mu[4 * 64]; acc = fma(d, d, acc);
    d = (double)bf16_hi(v.z) - mu[5 * 64]; acc = fma(d, d, acc);
    d = (double)bf16_lo(v.w) - mu[6 * 64]; acc = fma(d, d, acc);
    d = (double)bf16_hi(v.w) - mu[7 * 64]; acc = fma(d, d, acc);
}

// grid (ceil(N/rows_per_wg), B), block 512 (eight waves, two per SIMD to cover each other's fp64 chains), dynamic
// LDS = CH*512 doubles.  The mean (sum of the chunk partials / N) is staged in LDS as
// [group of 512 cols][j = col%8][lane = (col%512)/8] so that the 64 lanes of a wave read consecutive doubles.  A
// wave scores two tokens at a time; its first two tokens' loads go out before the mean is summed.
// CH: 512-column groups of a row (D <= 512*CH).
constexpr int kScoreThreads = 512;
constexpr int kScoreRowsPerPass = kScoreThreads / 64 * 2;
template <int CH>
__global__ __launch_bounds__(kScoreThreads) void score_kernel(const bf16_t* __restrict__ x,
                                                              const double* __restrict__ partial, int n_chunks,
                                                              float* __restrict__ score, int N, int D, int passes) {
    extern __shared__ double mu_s[];
    const int b = blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int n_first = blockIdx.x * passes * kScoreRowsPerPass + wave * 2;
    uint4 v0[CH], v1[CH];
    auto fetch = [&](int n0) {
        const bf16_t* row0 = x + ((size_t)b * N + min(n0, N - 1)) * D;
        const bf16_t* row1 = x + ((size_t)b * N + min(n0 + 1, N - 1)) * D;
#pragma unroll
        for (int g = 0; g < CH; ++g) {
            const int col = g * 512 + lane * 8;
            if (col < D) {
                v0[g] = *reinterpret_cast<const uint4*>(row0 + col);
                v1[g] = *reinterpret_cast<const uint4*>(row1 + col);
            }
        }
    };
    fetch(n_first);
    const double* pb = partial + (size_t)b * n_chunks * D;
    for (int c = threadIdx.x; c < D; c += kScoreThreads) {
        double a[kMaxChunks];
#pragma unroll
        for (int y = 0; y < kMaxChunks; ++y) a[y] = y < n_chunks ? pb[(size_t)y * D + c] : 0.0;
        double s = a[0];
#pragma unroll
        for (int y = 1; y < kMaxChunks; ++y) s += a[y];
        const int g = c >> 9, r = c & 511;
        mu_s[g * 512 + (r & 7) * 64 + (r >> 3)] = s / (double)N;
    }
    __syncthreads();
    for (int ps = 0; ps < passes; ++ps) {
        const int n0 = n_first + ps * kScoreRowsPerPass;
        if (n0 >= N) return;
        double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
        for (int g = 0; g < CH; ++g) {
            if (g * 512 + lane * 8 < D) {
                const double* mu = mu_s + g * 512 + lane;
                sqdev8(acc0, v0[g], mu);
                sqdev8(acc1, v1[g], mu);
            }
        }
        if (ps + 1 < passes) fetch(n0 + kScoreRowsPerPass);
        acc0 = wave_sum(acc0);
        acc1 = wave_sum(acc1);
        if (lane == 0) {
            score[(size_t)b * N + n0] = (float)acc0;
            if (n0 + 1 < N) score[(size_t)b * N + n0 + 1] = (float)acc1;
        }
    }
}

// Order-preserving map of an fp32 bit pattern to an unsigned key.
__device__ __forceinline__ uint32_t float_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

// Set bits of a wave mask below this lane's own.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

constexpr int kTopkThreads = 1024;
constexpr int kTopkWaves = kTopkThreads / 64;
constexpr int kBins = 1024;      // one per thread
constexpr int kBinCopies = 8;
constexpr int kMaxCand = 256;

// grid (B), block 1024, 0 < k < N <= 1024*E: wave w owns the 64*E tokens from w*64*E on, lane l of it every 64th of
// them (loads and stores are contiguous over a wave), with the keys in registers.
//   1. smallest and largest key; the range between them is cut into at most 1024 equal bins (a power of two wide)
//   2. histogram, one scan for the bin that holds the k-th largest key
//   3. that bin usually holds a few keys: they are ranked against each other directly.  If it holds more than
//      256, its range is cut into bins again (a map of equal scores ends with bins one key wide).
//   4. ordered compaction of the kept tokens (ties to the lowest index)
// Equal-width bins over the keys' own range spread the scores of a map over hundreds of bins, so the histogram's
// LDS atomics seldom meet and one pass nearly always leaves a few candidates; 8-bit digits below the common
// leading bits piled a whole wave onto a handful of bins and took three to four passes.  Neighbouring tokens of a
// smooth map still have neighbouring scores: every bin has eight counters in different banks, one per lane % 8
// (the launch inside the step: 4096 scores 10.3 -> 6.8 us, 16384 scores 29 -> 15).  Beyond 16384 tokens (E = 32) a few registers
// spill; 32761 tokens, whole selection: 119 -> 75 us all the same.
template <int E>
__global__ __launch_bounds__(kTopkThreads) void topk_kernel(const float* __restrict__ score, int N, int k,
                                                            int32_t* __restrict__ idx,
                                                            int32_t* __restrict__ rank) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins * kBinCopies];   // bin r: keys of the r-th highest range
    __shared__ uint32_t wave_a[kTopkWaves], wave_b[kTopkWaves];
    __shared__ uint32_t sel[3];
    __shared__ uint32_t cand[kMaxCand];
    __shared__ uint32_t n_cand;

    const int b = blockIdx.x;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const int n0 = wave * (64 * E) + lane;       // token of register j: n0 + 64*j
    const float* sc = score + (size_t)b * N;
    uint32_t key[E];
#pragma unroll
    for (int j = 0; j < E; ++j) key[j] = n0 + 64 * j < N ? max(float_key(sc[n0 + 64 * j]), 1u) : 0u;   // 0: no token
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        kmin = min(kmin, key[j] - 1u);
        kmax = max(kmax, key[j]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o, 64));
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o, 64));
    }
    if (lane == 0) { wave_a[wave] = kmin; wave_b[wave] = kmax; }
    __syncthreads();
#pragma unroll
    for (int wv = 0; wv < kTopkWaves; ++wv) { kmin = min(kmin, wave_a[wv]); kmax = max(kmax, wave_b[wv]); }
    kmin += 1u;

    // ---- T = key of the k-th largest, need = how many keys equal to T are kept
    uint32_t T, need, k_rem = (uint32_t)k;
    for (;;) {
        const uint32_t range = kmax - kmin;
        const int shift = range < (uint32_t)kBins ? 0 : 32 - __clz(range) - 10;     // range >> shift < 1024
        static_assert(kBins == 1024 && kBins == kTopkThreads && kBinCopies == 8, "ten bits of bin index, a thread per bin");
        reinterpret_cast<uint4*>(hist)[t] = make_uint4(0, 0, 0, 0);
        reinterpret_cast<uint4*>(hist)[t + kTopkThreads] = make_uint4(0, 0, 0, 0);
        if (t == 0) n_cand = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (key[j] - kmin <= kmax - kmin)
                atomicAdd(&hist[(kBins - 1 - ((key[j] - kmin) >> shift)) * kBinCopies + (lane & 7)], 1u);
        __syncthreads();
        const uint4 ha = reinterpret_cast<const uint4*>(hist)[2 * t], hb = reinterpret_cast<const uint4*>(hist)[2 * t + 1];
        const uint32_t here = ((ha.x + ha.y) + (ha.z + ha.w)) + ((hb.x + hb.y) + (hb.z + hb.w));
        uint32_t incl = here;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t v = __shfl_up(incl, o, 64);
            if (lane >= o) incl += v;
        }
        if (lane == 63) wave_a[wave] = incl;
        __syncthreads();
        uint32_t before = incl - here;
#pragma unroll
        for (int wv = 0; wv < kTopkWaves; ++wv) before += wv < wave ? wave_a[wv] : 0u;
        if (before < k_rem && k_rem <= before + here) { sel[0] = t; sel[1] = k_rem - before; sel[2] = here; }
        __syncthreads();
        const uint32_t count = sel[2];
        kmin += (uint32_t)(kBins - 1 - sel[0]) << shift;
        kmax = min(kmax - kmin, (1u << shift) - 1u) + kmin;   // (the highest bin may reach past the largest key)
        k_rem = sel[1];
        if (shift == 0) { T = kmin; need = k_rem; break; }
        if (count <= kMaxCand) {
#pragma unroll
            for (int j = 0; j < E; ++j)
                if (key[j] - kmin <= kmax - kmin) cand[atomicAdd(&n_cand, 1u)] = key[j];
            __syncthreads();
            if (t < (int)count) {
                const uint32_t mine = cand[t];
                uint32_t above = 0, equal = 0;
#pragma unroll 8
                for (uint32_t i = 0; i < count; ++i) {
                    const uint32_t c = cand[i];
                    above += c > mine ? 1u : 0u;
                    equal += c == mine ? 1u : 0u;
                }
                if (above < k_rem && k_rem <= above + equal) { sel[0] = mine; sel[1] = k_rem - above; }
            }
            __syncthreads();
            T = sel[0];
            need = sel[1];
            break;
        }
    }

    // ---- ordered compaction
    uint32_t total = 0;  // (greater << 16) | equal ; both at most 32768
#pragma unroll
    for (int j = 0; j < E; ++j) total += (key[j] > T ? 0x10000u : 0u) + (key[j] == T ? 1u : 0u);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) total += (uint32_t)__shfl_xor((int)total, o, 64);
    if (lane == 0) wave_b[wave] = total;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int wv = 0; wv < kTopkWaves; ++wv) before += wv < wave ? wave_b[wv] : 0u;
    // the first tokens equal to T, in order, are kept until `need` of them are
    uint32_t kept = (before >> 16) + min(before & 0xFFFFu, need), eq_seen = before & 0xFFFFu;
    const bool has_eq = __any((total & 0xFFFFu) != 0u) && eq_seen < need;
    int32_t* const idx_b = idx + (size_t)b * k;
    int32_t* const rank_b = rank ? rank + (size_t)b * N : nullptr;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int n = n0 + 64 * j;
        bool keep = key[j] > T;
        if (has_eq) {
            const uint64_t m_eq = __ballot(key[j] == T);
            keep = keep || (key[j] == T && eq_seen + lanes_below(m_eq) < need);
            eq_seen += (uint32_t)__popcll(m_eq);
        }
        const uint64_t m = __ballot(keep);
        const int pos = (int)(kept + lanes_below(m));
        kept += (uint32_t)__popcll(m);
        if (keep) idx_b[pos] = n;
        if (rank_b && n < N) rank_b[n] = keep ? pos : -1;
    }
}

// Every token kept (all = true): idx and rank are the identity; none kept: rank is -1 everywhere.
__global__ __launch_bounds__(256) void trivial_selection_kernel(int N, long total, bool all, int32_t* __restrict__ idx,
                                                                int32_t* __restrict__ rank) {
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int n = (int)(i % N);
    if (all) idx[i] = n;
    if (rank) rank[i] = all ? n : -1;
}

}  // namespace

SelectPlan select_plan(int B, int N, int D) {
    SelectPlan p;
    const int chunks = column_chunks(N, D);
    p.rows_per_chunk = ((N + chunks - 1) / chunks + kColRows - 1) / kColRows * kColRows;
    p.n_chunks = (N + p.rows_per_chunk - 1) / p.rows_per_chunk;
    // The size of the area is part of the interface (callers keep buffers of it, and the static entry point
    // accepts what fits into its array): partial sums of 32-row chunks, at most 256 of them, then mean and scores.
    // The kernels use the head of the first part and the scores.
    int rows = 32;
    while ((N + rows - 1) / rows > 256) rows *= 2;
    size_t off = 0;
    p.off_partial = off;
    off += (size_t)B * ((N + rows - 1) / rows) * D * sizeof(double);
    off += (size_t)B * D * sizeof(double);
    p.off_score = off;
    off += (((size_t)B * N * sizeof(float)) + 255) & ~(size_t)255;
    p.bytes = (off + 255) & ~(size_t)255;
    return p;
}

void launch_keep_all(int32_t* idx, int B, int N, hipStream_t stream) {
    const long total = (long)B * N;
    trivial_selection_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(N, total, true, idx, nullptr);
}

void launch_select(const void* x, int B, int N, int D, int k, int32_t* idx, int32_t* rank, float* score_out,
                   void* ws, const SelectPlan& plan, hipStream_t stream) {
    const bool trivial = k == 0 || k == N;
    if (trivial && (k > 0 || rank)) {
        const long total = (long)B * N;
        trivial_selection_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(N, total, k > 0, idx, rank);
    }
    if (trivial && !score_out) return;
    char* w = static_cast<char*>(ws);
    double* partial = reinterpret_cast<double*>(w + plan.off_partial);
    float* score = score_out ? score_out : reinterpret_cast<float*>(w + plan.off_score);
    const bf16_t* xb = static_cast<const bf16_t*>(x);

    colsum_kernel<<<dim3((D + kColTile - 1) / kColTile, plan.n_chunks, B), 256, 0, stream>>>(
        xb, partial, N, D, plan.rows_per_chunk, plan.n_chunks);
    // one pass of 16 tokens per workgroup while that gives few workgroups; the mean is summed once per workgroup,
    // so beyond two rounds of them (two fit a CU) a workgroup takes more passes
    int passes = 1;
    while (passes < 8 && (long)B * ((N + passes * kScoreRowsPerPass - 1) / (passes * kScoreRowsPerPass)) > 512) passes *= 2;
    const dim3 sgrid((N + passes * kScoreRowsPerPass - 1) / (passes * kScoreRowsPerPass), B);
#define FV_SCORE_CASE(CHV)                                                                                 \
    score_kernel<CHV><<<sgrid, kScoreThreads, (size_t)CHV * 512 * sizeof(double), stream>>>(xb, partial,   \
                                                                                            plan.n_chunks, \
                                                                                            score, N, D, passes)
    const int ch = (D + 511) / 512;
    if (ch <= 1) FV_SCORE_CASE(1);
    else if (ch <= 2) FV_SCORE_CASE(2);
    else if (ch <= 4) FV_SCORE_CASE(4);
    else if (ch <= 8) FV_SCORE_CASE(8);
    else FV_SCORE_CASE(16);   // D <= 8192, checked by the caller
#undef FV_SCORE_CASE
    if (trivial) return;
#define FV_TOPK_CASE(EV) topk_kernel<EV><<<dim3(B), kTopkThreads, 0, stream>>>(score, N, k, idx, rank)
    if (N <= 1024) FV_TOPK_CASE(1);
    else if (N <= 2048) FV_TOPK_CASE(2);
    else if (N <= 4096) FV_TOPK_CASE(4);
    else if (N <= 8192) FV_TOPK_CASE(8);
    else if (N <= 16384) FV_TOPK_CASE(16);
    else FV_TOPK_CASE(32);   // N <= 32768, checked by the caller
#undef FV_TOPK_CASE
}

}  // namespace fv
