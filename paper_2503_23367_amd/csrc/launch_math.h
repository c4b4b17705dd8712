// Index and plan arithmetic of the launches, without any HIP type: host code, kernels and a plain C++ compiler take
// the same lines, so the arithmetic can be checked at sizes that no test would launch.
#pragma once

#if defined(__HIPCC__)
#define FV_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define FV_HOST_DEVICE inline
#endif

namespace fv {

// A launch that clears arrival counters on the side (ZeroCounters) lets its first workgroups do it: thread `thread` of
// workgroup `block` clears first, first + step, ...  Grids have up to 2^31 workgroups, so the flat thread index of all of
// them does not fit 32 bits; of the first 256 it does.
constexpr unsigned kClearBlocks = 256;
constexpr unsigned kClearThreads = 256;   // threads of such a workgroup
struct CounterShare {
    int first, step;
};
FV_HOST_DEVICE bool clears_counters(unsigned block) { return block < kClearBlocks; }
FV_HOST_DEVICE CounterShare counter_share(unsigned block, unsigned thread, unsigned blocks) {
    const unsigned used = blocks < kClearBlocks ? blocks : kClearBlocks;
    return {(int)(block * kClearThreads + thread), (int)(used * kClearThreads)};
}

// Products of few rows (skinny.hip): a workgroup of `waves` waves owns `cols` output columns over all of K, taken in
// turns of 64.  Sixteen columns fill a matrix operand; eight take two halves of K side by side, so a wave's turn
// covers two of K's.  A wave has `turns` of its turns in flight at a time.
constexpr int kFewRowsMax = 16;      // most rows: one 16x16 operand
constexpr int kFewRowsWaves = 8;
constexpr int kFewRowsTurns = 4;
constexpr int kFewRowsRound = 64 * kFewRowsWaves * kFewRowsTurns;   // K that eight waves have in flight (2048)
struct FewRowsPlan {
    int cols, waves, turns;
};
FV_HOST_DEVICE int few_rows_share(int K, int cols) { return cols == 8 ? (K / 64 + 1) / 2 : K / 64; }
// `layernorm`: a product that a LayerNorm can go in front of (QKV, FC1).  Up to one round of K it has one split of K
// whether the LayerNorm is in front or, with an index list, in the gather's launch: the results are the same bits.
FV_HOST_DEVICE FewRowsPlan few_rows_plan(int N, int K, bool layernorm) {
    FewRowsPlan p;
    p.cols = (layernorm && K <= kFewRowsRound) || (N >= 16 * 256 && N % 16 == 0) ? 16 : 8;
    p.waves = p.cols == 8 && K > kFewRowsRound ? 2 * kFewRowsWaves : kFewRowsWaves;
    // Loads are not in branches, so a wave whose turns are used up loads the last one again.  Turns in flight that
    // divide the share evenly over the rounds keep that to less than one turn a wave and round; always four of
    // them loaded 64 turns for 18 at K = 2304 (out-proj of four rows 9.4 us in the tiled product, 17.8 that way).
    const int share = few_rows_share(K, p.cols);
    const int rounds = (share + p.waves * kFewRowsTurns - 1) / (p.waves * kFewRowsTurns);
    p.turns = (share + p.waves * rounds - 1) / (p.waves * rounds);
    return p;
}

// Which product takes M rows: this one, or the tiled one of gemm.hip (split_k: which can split this K between
// workgroups).  Every workgroup reads the rows' operands again, so the gain falls with the rows and with the number of
// workgroups; and a K of several rounds waits for memory once a round, for longest where the last round is part-filled.
// us, tiled / this one, weights from memory:
//   one round, part-filled: K = 1024, 24576 columns of 8 rows 12.5 / 13.3, 32768 of one row 15.5 / 14.7;
//   full rounds: K = 2048, 16384 of 8 / 16 rows 19.8 / 17.3, 19.9 / 20.9; K = 4096, 16384 of 8 / 12 / 16 rows 38.6 / 31.4,
//     37.1 / 34.7, 38.8 / 38.2; K = 8192, 32768 of 1 / 8 rows 118 / 104, 119 / 115;
//   several, part-filled: K = 2304, 12288 of 8 / 16 rows 19.6 / 17.0, 19.6 / 20.4, 16384 of 1 / 8 rows 20.4 / 17.9,
//     20.5 / 21.9; K = 5120, 8192 of 16 rows 25.3 / 27.5;
//   against a split K, up to 2048 columns (a workgroup per CU): 1024 of K = 4096, 1 / 16 rows 11.3 / 7.9, 11.8 / 10.7;
//     1536 of 6144, 8 / 16 rows 13.2 / 12.0, 13.1 / 14.1;
//   beyond, only where every CU has the same number of workgroups of sixteen columns: 4096 of K = 4096, 1 / 16 rows 14.1 / 11.8,
//     14.4 / 13.9; 8192 of 8192, 4 / 8 rows 34.8 / 34.4, 35 / 38; but 2304 of 9216, 1 / 16 rows 17 / 26, 18 / 41, and 5120
//     of 20480, 2 rows 54 / 58.
FV_HOST_DEVICE bool few_rows_product(int M, int N, int K, bool split_k) {
    if (M > kFewRowsMax) return false;
    const bool full = K % kFewRowsRound == 0;
    if (split_k && K > kFewRowsRound)
        return N <= 2048 ? M <= 8 || K <= 2 * kFewRowsRound
                         : full && N % (16 * 256) == 0 && (M <= 4 || K <= 2 * kFewRowsRound);
    if (full) return M <= 8 || N <= (M <= 12 ? 16384 : 12288);
    if (K < kFewRowsRound) return M == 1 || N <= (M <= 8 ? 16384 : 12288);
    return N <= (M == 1 ? 16384 : M <= 8 ? 12288 : 2048);
}
// The `split_k` of a block's products, which have scratch for slices.
FV_HOST_DEVICE bool few_rows_tiled_splits(int N, int K) { return K >= 2048 && K / 64 % 2 == 0 && N <= 8192; }
// A LayerNorm over K columns fits in front: a wave holds its share of the rows in registers.
FV_HOST_DEVICE bool few_rows_layernorm(int M, int N, int K) {
    return K <= kFewRowsRound && few_rows_product(M, N, K, false);
}

// How much of a list of matrices (bytes[0], bytes[1], ..., in the order they are read) a launch of about `us` microseconds
// fetches ahead on its `idle` CUs, and on how many of them.  Whole matrices, as many as come in while the launch runs: 45 KB a
// microsecond and CU, 5.6 MB for the chip.  No more CUs than that takes: the launch's own loads wait behind the others.
// `cut`: products of few rows, whose columns are streamed by workgroups on their own, also gain from the first part of a matrix;
// their launches are short, so less of it and from more CUs.  Eight blocks of the large model, without / with, us: one row
// 327 / 318, 64 rows 473 / 450, 256 rows 707 / 675, 576 rows 1063 / 1005; one matrix more than this takes or one less: 64 rows
// 497 / 482, 256 rows 712 / 682, 576 rows 1037 / 1023; 64 rows on 64 and 256 CUs instead of 128: 498 / 473.
struct PrefetchPlan {
    long bytes;
    int blocks;
};
FV_HOST_DEVICE PrefetchPlan prefetch_plan(const long* bytes, int n, int idle, double us, bool cut) {
    const double per_cu = (cut ? 16.0e3 : 45.0e3) * us, all = idle * per_cu, chip = (cut ? 2.0e6 : 5.6e6) * us;
    const long budget = (long)(all < chip ? all : chip);
    PrefetchPlan p{0, 0};
    for (int i = 0; i < n; ++i) {
        const long left = budget - p.bytes, take = bytes[i] <= left ? bytes[i] : cut ? left : 0;
        p.bytes += take;
        if (take < bytes[i]) break;
    }
    if (p.bytes >= 128) p.blocks = ((int)(p.bytes / per_cu) + 16) / 16 * 16;
    if (p.blocks > idle / 8 * 8) p.blocks = idle / 8 * 8;
    if (p.blocks <= 0) p = PrefetchPlan{0, 0};
    return p;
}

// Row chunks of the selection's column sums, of a map of N tokens and D columns: in powers of two, as few as give the
// launch a workgroup per CU (64 columns each; 240 of the 256 count as all), none shorter than the 256 rows that a workgroup
// has in flight.  A function of the map alone, so that a sample's scores have the same bits in every batch.
// Batches have workgroups enough with fewer chunks, which every workgroup of the score launch adds up: one to four times
// 4096 x 2048 19.0 us with eight chunks, 19.4 with four; eight times 53.8 against 53.3, and 51.2 with one; 1024 x 1920 eight
// times 22.6 with four, 25.4 with eight.
constexpr int kColTile = 64;        // columns of a workgroup
constexpr int kMaxChunks = 16;
constexpr int kMinChunkRows = 256;
FV_HOST_DEVICE int column_chunks(int N, int D) {
    const int tiles = (D + kColTile - 1) / kColTile;
    int chunks = 1;
    while (chunks < kMaxChunks && tiles * chunks < 240 && N >= 2 * chunks * kMinChunkRows) chunks *= 2;
    return chunks;
}

}  // namespace fv
