// Index and plan arithmetic of the launches, without any HIP type: host code, kernels and a plain C++ compiler take
// the same lines, so the arithmetic can be checked at sizes that no test would launch.
#pragma once

#include <stddef.h>

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

// Columns of a workgroup of a product with a LayerNorm in front: of sixteen and twelve, what leaves the busiest CU fewer weights to pull in.
// Eight blocks of the large model, whose QKV is 384 workgroups of sixteen and 512 of twelve, 1 / 16 rows 278.3 / 272.2, 368.7 / 363.5 us, of the 512 px
// model 268.1 / 262.8 (one row).
FV_HOST_DEVICE int few_rows_columns(int N) {
    const auto busiest = [&](int cols) { return ((N + cols - 1) / cols + 255) / 256 * cols; };
    return busiest(12) < busiest(16) ? 12 : 16;
}
// The rows of a product without a LayerNorm in front go through LDS where all of them fit beside the sums (us, weights from memory,
// without / with: 1 / 4 / 8 rows of 2048 x 8192 10.7 / 8.2, 11.5 / 9.3, 12.1 / 10.4, of 1920 x 7680 10.4 / 7.8, 11.1 / 8.9, 11.9 / 9.9; 1 / 16 of 1024 x 4096 5.7 /
// 4.9, 8.5 / 7.1, of 2048 x 2048 4.4 / 4.1, 5.7 / 4.9, of 448 x 2048 4.2 / 3.8, 5.5 / 4.6; nothing in it at 448 x 448), whatever the number of
// workgroups, also where 128 KB leave a CU one of them: QKV of 12 / 16 rows of 12288 x 4096 25.2 / 24.3, 27.1 / 25.2, 12 / 16 rows of 8192 x 4096 17.5 /
// 16.4, 18.5 / 17.0, 12 of 16384 x 2048 17.1 / 15.0, 8 of 24576 x 2048 22.1 / 19.8, 1 / 8 of 16384 x 4096 24.3 / 23.4, 28.1 / 25.1, 1 of 8192 x 8192 30.4 /
// 29.3.  The exception is one row over exactly a round of K in front of GELU or QKV, on as many workgroups a CU: there every load of a wave is out at
// once, the row's behind the weights' (4096 / 12288 / 16384 / 24576 x 2048 5.4 / 5.65, 10.8 / 11.1, 13.3 / 13.8, 18.4 / 19.6; two rows 5.5 / 5.3, 11.0 / 10.7, 13.6 /
// 13.3, 18.9 / 19.3; one of 6144 x 2048 7.7 / 7.6, of 12288 x 1984 10.5 / 9.8).
constexpr int kFewRowsLds = 128 << 10;
FV_HOST_DEVICE bool few_rows_in_lds(int M, int N, int K, bool layernorm) {
    if (M == 1 && layernorm && K == kFewRowsRound && N % (16 * 256) == 0) return false;
    return (long)M * K * 2 <= kFewRowsLds;
}

// Which product takes M rows: this one, or the tiled one of gemm_tiles.h (split_k: which can split this K between
// workgroups).  Every workgroup reads the rows' operands again, so the gain falls with the rows and with the number of
// workgroups; and a K of several rounds waits for memory once a round, for longest where the last round is part-filled.
// us, tiled / this one, weights from memory:
//   one round, part-filled: K = 1024, 24576 columns of 8 rows 12.5 / 13.3, 32768 of one row 15.5 / 14.7;
//   full rounds: K = 2048, 16384 of 8 / 16 rows 19.8 / 17.3, 19.9 / 20.9; K = 4096, 16384 of 8 / 12 / 16 rows 38.6 / 31.4,
//     37.1 / 34.7, 38.8 / 38.2; K = 8192, 32768 of 1 / 8 rows 118 / 104, 119 / 115;
//   several, part-filled: K = 2304, 12288 of 8 / 16 rows 19.6 / 17.0, 19.6 / 20.4, 16384 of 1 / 8 rows 20.4 / 17.9,
//     20.5 / 21.9; K = 5120, 8192 of 16 rows 25.3 / 27.5;
//   against a split K, whose slices then met inside the product, up to 2048 columns (a workgroup per CU): 1024 of K = 4096, 1 / 16 rows 11.3 / 7.9, 11.8 / 10.7;
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
// The `split_k` of a block's products.  Out-proj and FC2 of these shapes are cut into slices where the tiled product takes them; QKV
// and FC1 are not, but run on 64x32 tiles, one or two workgroups a CU, and beat this product as well: block of 1 / 4 / 8 rows, tiled
// QKV / this one, 2304 wide 57.3 / 57.6, 59.5 / 60.4, 61.3 / 63.2 us, 2560 wide 56.1 / 55.7, 57.2 / 58.2, 57.5 / 60.5.
FV_HOST_DEVICE bool few_rows_tiled_splits(int N, int K) { return K >= 2048 && K / 64 % 2 == 0 && N <= 8192; }
// A LayerNorm over K columns fits in front: a wave holds its share of the rows in registers.
FV_HOST_DEVICE bool few_rows_layernorm(int M, int N, int K) {
    return K <= kFewRowsRound && few_rows_product(M, N, K, false);
}

// The wide tiles' ring (gemm_tiles.h, main loop): a hand-over to tile kt + 1 waits for that tile's loads and opens the window in which the
// A tile kt + sa and the W tile kt + stages are fetched, A's loads first; a window ends before the next hand-over.
// Stages of A: as many as of W where 160 KB hold them, else two.
constexpr int wide_stages_a(int bm, int bn, int bk, int stages) { return stages * (bm + bn) * bk * 2 <= (160 << 10) ? stages : 2; }
// Slots from one load to the next, at most four, such that a K tile's loads find a slot each: of its last k-step those behind the
// hand-over, of the others all.
constexpr int load_slots(int slots, int before, int ksteps, int loads) {
    for (int ls = 4; ls > 0; --ls)
        if ((slots - before + ls - 1) / ls + (ksteps - 1) * slots / ls >= loads) return ls;
    return 0;
}
// Loads of a window that the rest of the hand-over's own k-step issues.
constexpr int handover_loads(int slots, int before, int ls, int loads) {
    return (slots - before + ls - 1) / ls < loads ? (slots - before + ls - 1) / ls : loads;
}
// Loads that may still be out when the first tile is used: those of the other stages, and what the prologue issues of the first window.
constexpr int wide_out_at_start(int sa, int stages, int a_ld, int w_ld, int first_window) {
    return (sa - 2) * a_ld + (stages - 2) * w_ld + first_window;
}
// ... and at a hand-over with `left` tiles behind the current one: what was issued after the last load of the next tile.  With rings of
// one depth these are whole tiles, stages - 2 of them; with a shorter A ring the next tile's A is in the latest windows, and of it
// on W's loads of these may be out.
constexpr int wide_out_at_handover(int sa, int stages, int a_ld, int w_ld, int left) {
    const auto least = [](int a, int b) { return a < b ? a : b; };
    if (left < 1) return 0;
    if (sa == stages) return least(left - 1, stages - 2) * (a_ld + w_ld);
    const int w_tiles = left - (stages - sa);   // W tiles that exist from the window of the next tile's A on
    return least(left - 1, sa - 2) * a_ld + (w_tiles > 0 ? least(w_tiles, sa - 1) * w_ld : 0);
}

// Tile choice.  What the measurements on the block's shapes say:
//  * large products are limited by power and by what a tile's waves read from LDS: tiles of 160x128 and up on four waves, one a SIMD,
//    with the main loop's order written down (wide tiles in gemm_tiles.h).  Of the eight-wave tiles 128x128, 192x128 and 256x128 are
//    left: as fast up to there, and their epilogues, two waves a SIMD, are shorter.
//  * what is left is how evenly the tiles fill rounds of 256 workgroups; hence the many shapes.  The best of them beat the best of the
//    seven shapes before (all on 32x32x16 instructions) by 9 % on average over 691 products; the picks by 8 %: 2048 x 8192 x 2048 61.9 -> 56.6 us,
//    8192 x 2048 x 8192 222 -> 194, 2300 x 7680 x 1920 75 -> 65, 1200 x 7680 x 1920 48 -> 37, 2300 x 2048 x 8192 82.6 -> 73.2.
//  * a part-filled last round costs less than a full one (fewer workgroups share the memory system and the
//    power budget).
//  * shapes that give at most 128 tiles of 128x128 (few rows) are bound by what a CU pulls in (about 37 bytes a
//    nanosecond of what misses the L2, 110 of what hits it), so more workgroups on smaller tiles beat the better
//    operand reuse of the larger ones: 128x64 tiles with eight waves and six stages (four waves and three stages: 256 x 6144 x
//    2048 18.6 -> 16.6 us, 576 x 2048 x 2048 17.3 -> 14.0, 960 rows 18.3 -> 15.4), at most 64: 64x64 tiles with four stages, or
//    64x32 ones with eight where these are at most a round (64 x 6144 x 2048 13.2 -> 11.2, 25 rows 11.4 -> 9.3; 128 rows, a
//    round and a half, 13.1 -> 19.2) and K is more than four tiles: up to there the sums of their two k-groups, which meet in LDS, cost
//    more than the finer split saves (34 products 1 % longer; of K 320 to 512 3 % shorter with weights from memory, 1 % longer from
//    the cache, of K 576 to 1024 5 to 12 % shorter, of longer ones 16 to 50 %).  64x64 tiles with eight stages, one workgroup a
//    CU instead of two and all of a ring's loads queued in front of the first product, take 4 to 6 % longer with weights in the cache
//    (545 x 1024 x 1024 6.5 / 7.1 us, 350 x 2048 x 2048 9.1 / 9.9), and of K above 1024 2 to 8 % less with weights from memory
//    (68 x 5760 x 1920 12.5 / 11.5, 142 x 4096 x 4096 20.8 / 18.4): for QKV, whose weights no launch fetches ahead.
// Beyond 128 tiles the choice is the candidate with the least modelled time (us): 2.05 to launch, and for every round of its
// workgroups, a part-filled one counting 0.684 + 0.311 * fill, fix + K tiles * per_kt, where a K tile beyond the 32nd takes
// `longer` more; tile counts that do not divide by eight are not dealt to the XCDs in contiguous runs, and cost 4 % more, with
// three, five or seven tile rows 6 %.  The constants are a fit to 691 products (eight models' four products and generic ones; 65 to
// 16000 rows, N 128 to 24576, K 64 to 16384; weights from memory and from the cache) under each candidate, by the time that the picks
// lose: 1.3 % on the best of fifteen wide shapes and six others, of which these cost 0.7 % to have left out.
enum Tile {   // (of gemm_tiles.h)
    TILE_64x32 = 18, TILE_64x64 = 16, TILE_64x64_DEEP = 15, TILE_128x64 = 17, TILE_128x128 = 40, TILE_160x128 = 35, TILE_192x128 = 34,
    TILE_192x192 = 14, TILE_192x256 = 13, TILE_224x128 = 36, TILE_224x192 = 37, TILE_224x256 = 38, TILE_256x128 = 32, TILE_256x192 = 12,
    TILE_256x256 = 11
};
struct TileChoice {
    int cfg;
    double us;   // modelled
};
FV_HOST_DEVICE double tile_rounds(int M, int N, int bm, int bn, int slots, int splits, double part, double fill, double uneven,
                                  double scattered) {
    const long tile_rows = (M + bm - 1) / bm, tiles = tile_rows * ((N + bn - 1) / bn);
    const long full = tiles * splits / slots, rem = tiles * splits - full * slots;
    const double rounds = (double)full + (rem ? part + fill * (double)rem / slots : 0.0);
    return tiles % 8 == 0 ? rounds : rounds * (1.0 + (tile_rows == 3 || tile_rows == 5 || tile_rows == 7 ? scattered : uneven));
}
FV_HOST_DEVICE TileChoice gemm_choose_tile(bool qkv, int M, int N, int K) {
    const long tiles128 = (long)((M + 127) / 128) * ((N + 127) / 128);
    const int KT = K / 64;
    struct Cand { int cfg, bm, bn, slots; double fix, per_kt, longer; };
    const Cand cands[] = {
        // the first three by the rules above, their times for the K slices below, with round factors of their own: under those of the wide
        // tiles they came out a microsecond short, and out-proj of 260 to 450 rows stayed whole (block of 259 / 286 rows 1920 wide 92.2 / 95.2 us,
        // in two slices 90.8 / 94.0; stacks of eight blocks of 14x21 tokens 749 us 1920 wide, 761 whole, 874 and 890 2304 wide)
        {TILE_64x32, 64, 32, 256, 2.1, 0.170, 0.0},
        {qkv && KT > 16 ? TILE_64x64_DEEP : TILE_64x64, 64, 64, 512, 2.7, 0.270, 0.0},
        {TILE_128x64, 128, 64, 256, 3.4, 0.335, 0.0},
        {TILE_128x128, 128, 128, 256, 3.33, 0.500, -0.023},
        {TILE_160x128, 160, 128, 256, 4.50, 0.582, -0.016},
        {TILE_192x128, 192, 128, 256, 3.94, 0.670, -0.002},
        {TILE_192x192, 192, 192, 256, 6.51, 0.891, -0.048},
        {TILE_192x256, 192, 256, 256, 9.22, 1.076, -0.045},
        {TILE_224x128, 224, 128, 256, 6.42, 0.689, -0.021},
        {TILE_224x192, 224, 192, 256, 8.80, 0.938, -0.027},
        {TILE_224x256, 224, 256, 256, 10.46, 1.251, -0.018},
        {TILE_256x128, 256, 128, 256, 5.15, 0.864, 0.008},
        {TILE_256x192, 256, 192, 256, 8.69, 1.055, -0.013},
        {TILE_256x256, 256, 256, 256, 11.57, 1.367, 0.034},
    };
    int from = 3, to = (int)(sizeof(cands) / sizeof(cands[0]));
    if (tiles128 <= 64) from = (long)((M + 63) / 64) * ((N + 31) / 32) <= 256 && KT > 4 ? 0 : 1;
    else if (tiles128 <= 128) from = 2;
    if (from < 3) to = from + 1;
    TileChoice best{TILE_128x128, 1e30};
    for (int i = from; i < to; ++i) {
        const Cand& c = cands[i];
        const double rounds = i < 3 ? tile_rounds(M, N, c.bm, c.bn, c.slots, 1, 0.777, 0.189, 0.037, 0.10)
                                    : tile_rounds(M, N, c.bm, c.bn, c.slots, 1, 0.684, 0.311, 0.041, 0.062);
        const double t = 2.05 + rounds * (c.fix + KT * c.per_kt + (KT > 32 ? (KT - 32) * c.longer : 0.0));
        if (t < best.us) best = TileChoice{c.cfg, t};
    }
    return best;
}

// Plan of an out-proj or FC2 product of few rows: the K range is cut into `splits` slices that run as separate workgroups
// and leave fp32 sums [splits][M][N] in scratch; splits == 1: no scratch needed.
struct SplitKPlan {
    int splits = 1;
    int cfg = 0;        // tile of the slices (gemm_sliced.hip)
    size_t bytes = 0;
};
// What the slices meet in.  A LayerNorm of the rows that follows anyway (out-proj of a whole block) adds them up for next to
// nothing; where none does (a half of a block on its own), a launch of its own does, 3.6 us.  FC2 of a block has a LayerNorm
// behind it in a stack and none in a single step; both use one plan, so that a stack has the bits of its single blocks: half.
enum SlicesMeet { MEET_IN_LAYERNORM = 0, MEET_IN_EITHER = 1, MEET_IN_LAUNCH = 2 };
// Whether the K of such a product is cut, and on which tile.  Few output tiles leave CUs idle and make each of the others walk
// all of K; slices fill the chip, at the price of their sums going through memory.  The candidate with the least modelled time (us): 2.2 to
// launch; a round of 256 workgroups at fix + K tiles of a slice * per_kt, a part-filled one 0.804 + 0.156 * fill, 3 % more where
// the tiles do not divide evenly among the XCDs, 21 % with three, five or seven tile rows; 0.505 for every MB of slices; and the
// meeting.  Against it the whole product at its tile's modelled time.  The constants are a fit to 480 products of seven models, 17 to 2600
// rows, inside the calls that run them, on 32x32x16 instructions; on today's kernels, in 540 blocks and their halves (seven widths, the same rows), the
// picks lose 0.05 (out-proj on its own) to 0.33 us (FC2 on its own) a product on the best candidate, with the meeting raised from 1.5 to 1.8.  A new fit of all
// constants lost 0.05 to 0.31 and was up to 3 % slower on blocks that these pick right.  A fit
// to 30 products of the large model lost 0.3 to 0.9, most of it in halves on their own, whose sum it took for free (attention
// half of 357 rows 2304 wide 56.1 us, whole 51.0; of 443 rows of the small model 30.1 / 27.1), and at seven tile rows
// (MLP half, 813 rows 1920 wide: two slices on 128x128 tiles 82.9, whole 78.8).  160x128 tiles in four slices are not offered: they win on 20 of 1002
// products, around a full round (FC2 of 560 to 640 rows 1920 and 2048 wide, 1 to 8 us), and lose 4 us on the middle one.
FV_HOST_DEVICE SplitKPlan gemm_splitk_plan(int M, int N, int K, SlicesMeet meet) {
    SplitKPlan best;
    if (few_rows_product(M, N, K, few_rows_tiled_splits(N, K))) return best;   // skinny.hip
    struct Cand { int cfg, bm, bn, max_splits; double fix, per_kt; };
    const Cand cands[] = {{TILE_64x64, 64, 64, 8, 0.94, 0.244}, {TILE_128x64, 128, 64, 4, 2.07, 0.293},
                          {TILE_128x128, 128, 128, 4, 1.5, 0.492}, {TILE_160x128, 160, 128, 2, 2.43, 0.555},
                          {TILE_192x128, 192, 128, 4, 1.55, 0.638}};
    const int KT = K / 64;
    double least = gemm_choose_tile(false, M, N, K).us;
    for (const Cand& c : cands)
        for (int s = 2; s <= c.max_splits; s *= 2) {
            const long tiles = (long)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
            if (KT % s != 0 || KT / s < 4 || tiles * s > 256) continue;
            const double t = 2.2 + tile_rounds(M, N, c.bm, c.bn, 256, s, 0.804, 0.156, 0.033, 0.214) * (c.fix + KT / s * c.per_kt) +
                             4.0e-6 * s * M * N * 0.505 + 1.8 * meet;
            if (t < least) {
                least = t;
                best.splits = s;
                best.cfg = c.cfg;
                best.bytes = (size_t)s * M * N * 4;
            }
        }
    return best;
}

// Attention without key ranges: which kernel and workgroups (attention.hip), of B samples, H heads of dim dh, k queries, L keys.
// Head dim 128 and more than two key tiles: the software-pipelined kernel (64 queries per wave), with 128-query workgroups (5: two
// query groups x two key slices) or 256-query workgroups (6: four query groups), whichever needs less time for its rounds
// of workgroups on 256 CUs; a 256-query workgroup does twice the work about 7 % faster.  The plain kernel (a wave per 32 queries)
// otherwise, on workgroups as small as still fit a round: there the launch waits for its keys, which more CUs then pull on, a block's
// time in us:
//   2: one tile of 64 keys: nothing to split, 128 queries (37.9 for one token of the large model, 40.0 with 128-key tiles);
//   7: head dim 128, up to 176 workgroups of 32 queries, keys split in two: 256 queries over 521 keys 79.7 (64 queries: 81.1),
//     300 over 1221 117.1 (118.9); 208 workgroups of them lose (400 over 921 104.5, 102.4).  Up to 32 queries there are as many
//     workgroups of 64, whose second query group only loads, and two waves that load keys lose to four until the cache is long:
//     the launch over 300 / 600 / 1200 / 2500 keys 9.4 / 12.0 / 17.5 / 28 us on two waves, 8.9 / 11.7 / 17.3 / 30 on four.
//     Nor where workgroups of 64 divide evenly among the eight XCDs and those of 32 do not, so that every XCD pulls in every
//     head's keys (18 heads, 222 over 1103 keys 18.8, 17.0 on 64);
//   3: up to 256 workgroups of 64 queries, keys split in two: small model, 576 over 1497 62.9, 1024 over 2624 88.3 (128 queries on
//     eight waves: 67.3, 92.3), 4 x 169 of the large model over 424 123.7 (pipelined: 130); 270 of them lose (576 over 1497 of
//     the 512 px model 129.8, 126.4);
//   more: with enough queries two 4-wave workgroups of 128 share a CU (2); with fewer an 8-wave workgroup splits the
//     keys of each tile between two waves per query group (4).
FV_HOST_DEVICE int attention_cfg(int B, int H, int dh, int k, int L) {
    const auto groups = [&](int queries) { return (long)((k + queries - 1) / queries) * H * B; };
    const long wg256 = groups(256), wg128 = groups(128), wg64 = groups(64), waves = groups(32);
    // Head dim 64 is bound by the softmax, not the matrix pipe, and the pipelined kernel gains less: its 256-query workgroups
    // win (by 5-20 % on 8 x 30 heads, 1024-3072 keys) where they pad the queries no further than 128-query workgroups would
    // and the key loop is long enough to pay for the longer prologue; the plain kernel wins elsewhere.
    if (dh == 64 && L >= 1024 && wg256 >= 128 && (k + 255) / 256 * 2 == (k + 127) / 128) return 6;
    if (L <= 64) return 2;
    if (dh == 128 && waves <= 176) return (k > 32 || L > 1536) && (waves % 8 == 0 || wg64 % 8 != 0) ? 7 : 3;
    if (wg64 <= 256 && (dh == 64 || wg128 < 128 || L <= 512)) return 3;
    if (dh == 128 && L > 256) {
        const long rounds128 = (wg128 + 255) / 256, rounds256 = (wg256 + 255) / 256;
        return 1.86 * (double)rounds256 < (double)rounds128 ? 6 : 5;
    }
    return waves >= 1800 ? 2 : 4;
}

// Head dim 64 on workgroups of 64 queries with a tile's keys split in two (3 above): over longer caches on what it runs instead.  Tiles
// of 256 keys split between four waves halve the turns that a wave waits for its keys, and hold twice the keys in flight (128 KB a
// workgroup; head dim 128 has no room for that).  us, two slices / four over 32 queries / four over 64, caches from memory, 16 heads: 100
// queries over 300 / 500 / 600 / 700 / 1000 / 1300 / 2600 keys 6.6 / 8.9 / 9.9 / 10.4 / 13.6 / 16.7 / 24.5, 7.3 / 8.7 / 9.7 / 9.6 / 11.9 / 14.5 / 19.6, 8.2 / 9.3 / 10.7 / 10.6 / 12.6 / 15.8 /
// 21.9; 60 queries of 30 heads over 5000 48.8, 39.2, 40.2.  So four slices over 32 queries from 640 keys on, where their workgroups are at
// most half a round, which leaves CUs to fetch weights on, and divide among the XCDs if those of 64 do (200 of 30 heads over 1000 keys 13.5,
// 14.4, 12.6); else over 64 queries where tiles of 256 waste little (800 / 1000 / 2200 / 3500 keys 11.5 / 13.4 / 22.8 / 31.1, 12.2 / 12.6 / 19.6 /
// 25.8) and do not fall unevenly on the XCDs (320 of 30 heads over 1600 / 2200 keys 17.2 / 25.4, 17.9 / 22.7).  Not a matter of what
// the launch fetches: a stack has the bits of its single blocks.
struct AttentionSlices {
    int queries, slices;
};
FV_HOST_DEVICE AttentionSlices attention_slices(int B, int H, int k, int L) {
    const long wg32 = (long)((k + 31) / 32) * H * B, wg64 = (long)((k + 63) / 64) * H * B;
    if (L > 640 && wg32 <= 128 && (wg32 % 8 == 0 || wg64 % 8 != 0)) return AttentionSlices{32, 4};
    if (L > 7 * 128 && wg64 <= 256 && (wg64 % 8 == 0 || L > 2048)) return AttentionSlices{64, 4};
    return AttentionSlices{64, 2};
}

// Which matrices the attention launch of a call may fetch ahead: those that the call's later products read, in their order, and no
// others; a call that does not go on to the MLP half may hold placeholders for its weights.  Matrices under 16 MB only in a
// stack, and not for few rows (16 blocks of the small model on 169 rows 775 -> 734 us with it, but its single step on 128 rows
// 55.8 -> 56.4 and eight blocks of it on 16 rows 241 -> 246).
struct AheadList {
    int n;           // of out-proj, FC1, FC2: the first n
    long bytes[3];
};
FV_HOST_DEVICE AheadList ahead_list(int D, int F, int M, bool in_stack, bool ffn_follows) {
    const AheadList all{ffn_follows ? 3 : 1, {2L * D * D, 2L * D * F, 2L * D * F}};
    return all.bytes[1] >= 16L << 20 || (in_stack && M > kFewRowsMax) ? all : AheadList{0, {0, 0, 0}};
}

// How much of a list of matrices (bytes[0], bytes[1], ..., in the order they are read) a launch of about `us` microseconds
// fetches ahead on its `idle` CUs, and on how many of them.  Whole matrices, as many as pay: 45 KB a microsecond and
// CU, 5.6 MB for the chip (fitted, not a bandwidth: a CU pulls in about 37, and what is still on its way when the launch
// ends arrives while the next one starts).  No more CUs than that takes: the launch's own loads wait behind the others.
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

// Consecutive workgroups go to the eight XCDs in turn, each with its own L2.  A map is walked in shares of four waves with `rows` token rows
// each.  In runs, an XCD has a contiguous run of a sample's shares, so the rows of a cached map that neighbouring rows are blended from are
// fetched into one L2 and not into all.  Which XCD has which run moves on by one a sample: the last run is the short one, and by always
// the same XCD batches of small maps waited for the other seven (8 x 48x48 x 2048 32.6 -> 30.6 us, 8 x 13x20 x 4096 9.9 -> 9.7).
// Dealt in turn, shares come round to an XCD every 32 * rows tokens: where the width is near a multiple of that, the positions above and below one another are
// on one XCD already, and runs share clustered kept sets out unevenly (restoration, in turn / in runs: 64x95 x 2048 13.3 / 14.1 us, 96x96 17.1 / 17.6,
// 128x128 26.6 / 27.3; but 80x80 14.45 / 14.54, 2 x 90x47 16.6 / 15.4, in pairs 96x96 x 1024 11.7 / 10.8; steps of the large model, whose fill this is,
// 2 and 5 % of 96x96 tokens kept behind 11059 186.7 / 188.3, 220.8 / 221.9, of 128x96 behind 14745 213.8 / 215.3, 275.0 / 276.0; 15 % of 48x48 behind 2764 146.4 / 145.9,
// 13 % of 80x80 behind 7680 246.4 / 245.2; nothing in it for the small models).  Under eight shares an XCD the runs are too short to matter.
constexpr int kXcdShares = 64;
FV_HOST_DEVICE bool columns_on_one_xcd(int w, int rows) {
    const int period = 32 * rows, off = w % period;
    return w > period / 2 && (off < 2 * rows || off > period - 2 * rows);
}
FV_HOST_DEVICE bool shares_in_runs(int shares, int w, int rows) { return shares >= kXcdShares && !columns_on_one_xcd(w, rows); }
// Workgroups that walk a sample, and the share that workgroup `block` of them takes; a share past the last one is nothing to do.
FV_HOST_DEVICE int xcd_blocks(int shares, bool runs) { return runs ? (shares + 7) / 8 * 8 : shares; }
FV_HOST_DEVICE int xcd_share(int block, int shares, bool runs, int sample) {
    return runs ? ((block + sample) & 7) * ((shares + 7) / 8) + (block >> 3) : block;
}

// Rows that a wave of the restoration takes, of maps of `rows` tokens in all, w wide, D columns.  Rank, taps and store of a row
// wait for one another, so a wave a row while the chip has room for them all (us, a pair unrolled / one: 16x16 x 1024 5.5 / 4.9,
// 53x37 x 2048 8.4 / 6.0, 64x64 x 2048 9.0 / 8.1, 4 x 33x31 x 1920 10.6 / 8.6, 40x44 x 4096 14.4 / 9.4), wide rows for longer (73x67 x 2048
// 12.1 / 10.9, 8 x 24x24 x 1920 12.8 / 11.1, 75x70 x 1920 12.0 / 11.1).  Maps of more rows than that have a queue of waves either way, and a pair
// has two rows' loads in flight (81x82 x 448 5.6 / 6.2, 100x104 x 1024 11.7 / 11.9, 72x80 x 1024 7.4 / 7.7, 2 x 90x77 x 1920 23.6 / 24.6), except
// of 4096 columns, which fill a wave by themselves (62x105 23.3 / 21.9).  Wide rows gain from the pair while few of them are kept, whose
// copies have no rank-to-taps wait to share (10 / 50 / 80 % kept: 85x88 x 2048 14.5 / 15.7, 15.6 / 14.9, 15.4 / 14.3; 120x112 24.0 / 25.2, 25.6 / 24.0,
// 25.9 / 22.1; 80x80 10 / 60 % 14.0 / 14.5, 14.0 / 13.6): widths near a multiple of sixteen, those of most schedules, have a row a wave at every size.  Beyond 2^25 elements two rows, one after the other (90x90 x 8192 a pair 54.4, one row 52.7, two 51.4; 8 x 100x100 x 1920
// 154.6, 145.0, 144.7).  All with shares in runs; dealt in turn, these plans' times were 2x90x77 x 1920 29.7 us (23.6 in
// runs), 100x120 x 4096 47.9 (39.6), 90x90 x 8192 68.4 (51.4), 40x44 x 4096 10.6 (9.4).
struct RestorePlan {
    int rows;
    bool pair;   // unrolled
};
FV_HOST_DEVICE RestorePlan restore_plan(long rows, int w, int D) {
    if (rows * D >= 1L << 25) return RestorePlan{2, false};
    if (rows < 4300 || D >= 4096 || (D >= 1280 && (rows < 6000 || (w + 1) % 16 <= 2))) return RestorePlan{1, false};
    return RestorePlan{2, true};
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
