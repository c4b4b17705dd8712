// bf16 MFMA GEMM for the block's four dense contractions (QKV, out-proj, FC1,
// FC2):  C[m,n] = sum_k A[m,k] * W[n,k]  with A [M,K] and W [N,K] both
// K-contiguous (activations are row-major, weights are [out, in]).
//
// Tiling for gfx950: a workgroup of 4 or 8 waves owns a BM x BN tile of C; each
// wave owns a sub-tile built from 16x16x32 bf16 MFMAs with fp32 accumulators.
// K is walked in tiles of BK: both operand tiles are copied global -> LDS by
// direct-to-LDS loads into a ring of STAGES stages (the next tiles' loads are in
// flight while the current one is multiplied), in rows whose 16-byte chunks are
// XOR-swizzled with the row index so that the MFMA operand reads (one 16-byte
// ds_read per lane, 16 consecutive rows per quarter of a wave) are conflict free.
//
// Why 16x16x32 and not 32x32x16 instructions: under this load the chip is limited by power, not by issue, and the smaller one moves half
// the accumulator bytes per operation.  One wave a SIMD on N(0, 1) data, nothing but matrix instructions: 1.73 PFLOP/s against
// 1.53 (on zeros both 2.17).  Products, same tiles: 2048 x 8192 x 2048 62.2 -> 57.6 us, 4096 x 8192 x 2048 120 -> 111.5, 256 x 8192 x 2048
// 14.5 -> 13.4; few-tile products of long K, which wait for memory, are within 2 % either way.
//
// Epilogues are fused: bias, residual add, GELU, and for the QKV GEMM the
// split into the query buffer and the append into the K / V caches
// (V transposed so that cache positions are contiguous).
#pragma once

#include <stdio.h>
#include <stdlib.h>

#include <mutex>
#include "common.h"
#include "kernels.h"

namespace fv {

struct GemmParams {
    const bf16_t* A;
    const bf16_t* W;
    const bf16_t* bias;
    int M, N, K;
    bf16_t* out;
    const bf16_t* residual;
    const int32_t* res_rows;  // optional row gather for the residual: row of output row m is res_rows[m]
    const int32_t* out_rows;  // optional row scatter of the output (EPI_BIAS_RES): row m goes to row out_rows[m]
    bf16_t* q_out;
    bf16_t* k_cache;
    bf16_t* v_cache;
    int D, H, dh, k_tokens, L0, L_cap;
    const float* rope_cos;     // optional [rope_N, dh/2] tables: q and the new keys are turned in the epilogue
    const float* rope_sin;
    const int32_t* rope_rows;  // slot of output row m = rope_rows[m] % rope_N (NULL: its token index)
    int rope_N;
    int tiles_m, tiles_n;
    int splits;        // K slices (grid.y); 1 unless the kernel is instantiated with SLICED
    float* slices;     // [slice][M][N] fp32 sums of the slices (SLICED)
};
// One file for each epilogue, since the kernels take long to compile: gemm_<epilogue>.hip.
void launch_tiles_qkv(GemmParams& p, hipStream_t stream);
void launch_tiles_rope(GemmParams& p, hipStream_t stream);
void launch_tiles_residual(GemmParams& p, hipStream_t stream);
void launch_tiles_gelu(GemmParams& p, hipStream_t stream);
void launch_tiles_sliced(const SplitKPlan& sk, GemmParams& p, hipStream_t stream);

// Tuning builds only (-DFASTVAR_DEV_KNOBS, never the product library, which reads no environment and keeps
// no state): FASTVAR_GEMM_CFG (all epilogues) or FASTVAR_GEMM_CFG<e> (epilogue e = 0, 1, 2) forces a tile
// configuration, unsliced; unset means gemm_choose_tile and gemm_splitk_plan.
inline int gemm_cfg_override(int epi) {
#ifdef FASTVAR_DEV_KNOBS
    char name[32];
    snprintf(name, sizeof(name), "FASTVAR_GEMM_CFG%d", epi);
    const char* e = getenv(name);
    if (!e) e = getenv("FASTVAR_GEMM_CFG");
    return e ? atoi(e) : -1;
#else
    (void)epi;
    return -1;
#endif
}

namespace {

// s_waitcnt immediate (gfx9 encoding): wait until at most `vm` vector-memory
// operations are outstanding; lgkm = true also waits for all LDS/scalar ops.
constexpr int waitcnt_imm(int vm, bool lgkm) {
    return (vm & 0xF) | ((vm >> 4) << 14) | (0x7 << 4) | ((lgkm ? 0x0 : 0xF) << 8);
}

// XOR key that spreads the 16-byte chunks of consecutive rows over all 64 LDS
// banks (256 bytes): a 16-byte-per-lane read is served 16 lanes at a time, so 16
// consecutive rows must land in 16 different chunk columns.  Rows of 128 bytes
// (8 chunks, two rows per bank sweep) use row bits 1-3.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

__device__ __forceinline__ f32x4_t mfma(const bf16x8_t& a, const bf16x8_t& b, const f32x4_t& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// WGM x WGN waves tile the BM x BN block; KG such groups of waves split every K
// tile between them (group g takes the g-th run of 32-wide k-steps) and are
// summed through LDS at the end.  Eight waves (two per SIMD) cover each other's
// barrier, load and LDS waits where the tile gives one wave per SIMD too little
// independent work.
// SLICED: the K range is also split between workgroups (blockIdx.y), each of which leaves the fp32 sums of its
// slice in scratch memory, row-major; the launch that follows adds the slices up (slice_sum_kernel in layernorm.hip),
// mostly the LayerNorm that reads the rows anyway.  The slices meeting inside this launch instead (partial tiles through
// memory, the last workgroup of a tile adding them up) cost every such product 3 to 8 us: FC2 of the large model at
// 64 / 256 / 576 / 1152 rows 13.3 / 25.2 / 43.2 / 60.2 us that way, 9.9 / 20.2 / 29.7 / 51.6 this way.
template <int EPI, int KG, bool SLICED, int BM, int BN>
constexpr bool kPersistent = !SLICED && KG == 1 && (is_qkv(EPI) || (EPI == EPI_BIAS_GELU && BM * BN >= 224 * 256));

// Wide tiles: 2 x 2 waves, one a SIMD, of at least 64x64 each.  A wave of 128x128 reads a third less from LDS per operation than
// one of 128x64, and has the registers for it (256 accumulators); nothing else hides its latencies, so the order of its
// instructions is the schedule and is written down slot by slot (the main loop).  256x256 on eight waves / this way: 2048 x 8192 of K
// 1024 / 2048 / 4096 / 8192 35.1 / 58.2 / 104.9 / 201 us, 35.8 / 57.3 / 99.2 / 187 (a K tile 1.51 us, 1.37; on 32x32x16 instructions and
// eight waves 1.61).  The A ring has as many stages as the W ring where 160 KB hold them, else two.
template <int BM, int BN, int WGM, int WGN, int KG>
constexpr bool kWide = WGM == 2 && WGN == 2 && KG == 1 && BM * BN >= 128 * 128;
template <int BM, int BN, int BK, int STAGES>
constexpr int kStagesA = wide_stages_a(BM, BN, BK, STAGES);

template <int BM, int BN, int BK, int STAGES, int WGM, int WGN, int KG, int EPI, bool SLICED = false>
__global__ __launch_bounds__(64 * WGM * WGN * KG) void gemm_nt_kernel(const GemmParams p) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass only needs the launch stub
    constexpr int NWQ = WGM * WGN;             // waves per k-group
    constexpr int NW = NWQ * KG;               // waves per workgroup
    constexpr int WTM = BM / WGM, WTN = BN / WGN;  // wave tile
    constexpr int MI = WTM / 16, NI = WTN / 16, NJ = WTN / 32;   // blocks of a matrix instruction; pairs of them along N
    constexpr int CPR = BK / 8;                // 16-byte chunks per LDS row
    constexpr int RPI = 64 / CPR;              // rows covered by one 64-lane direct-to-LDS load
    constexpr int KK = BK / 32 / KG;           // MFMA k-steps per tile and k-group
    constexpr int A_LD = BM / RPI / NW, W_LD = BN / RPI / NW;  // loads per wave per tile
    constexpr int LPT = A_LD + W_LD;
    constexpr int A_TILE = BM * CPR, W_TILE = BN * CPR;      // 16-byte chunks per stage
    constexpr int STAGE = A_TILE + W_TILE;
    static_assert(WTM % 16 == 0 && WTN % 32 == 0 && (BK / 32) % KG == 0, "wave tiles are made of pairs of 16x16x32 MFMAs");
    static_assert(A_LD * RPI * NW == BM && W_LD * RPI * NW == BN && NW % 2 == 0, "loads must tile the stage");
    // When a stage is refilled, one load per operand read.  EARLY, where k-groups leave a tile one k-step: at the hand-over that frees it.
    // Otherwise during the first k-step of the following tile, half a tile later, which is gentler on the hand-over.  (Wide tiles have their
    // own order, in the main loop.)
    static_assert(CPR == 8 && KK <= 2, "rows of 128 bytes, at most two k-steps a tile");
    constexpr bool EARLY = KK == 1;
    static_assert((STAGES - 1) * LPT <= 63, "vmcnt is 6 bits");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    u32x4_t* lds = reinterpret_cast<u32x4_t*>(smem);  // [STAGES][A tile | W tile]; wide tiles [SA][A tile] [STAGES][W tile]
    constexpr bool WIDE = kWide<BM, BN, WGM, WGN, KG>;
    constexpr int SA = kStagesA<BM, BN, BK, STAGES>;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / NWQ;                 // k-group
    const int wq = wave % NWQ;                 // position in the wave grid
    const int wm = wq / WGN, wn = wq % WGN;
    const int kk0 = kg * KK;                   // first k-step of this group inside a tile

    // Tile id: consecutive workgroup ids are dealt round-robin to the 8 XCDs;
    // undo that so each XCD (own L2) walks a contiguous run of tiles, and walk
    // tiles in groups of 8 tile-rows so neighbours share operand rows.
    // A QKV launch with more tiles than the chip holds workgroups at a time is persistent: the grid is one
    // round of workgroups, and workgroup i takes tiles i, i + grid, ... (the grid is a multiple of 8, so
    // a workgroup's tiles stay in its XCD's run).  What that buys is the overlap at the seam: the next
    // tile's first stages are fetched while this tile's epilogue runs, which needs no LDS.  It pays for the
    // QKV epilogue, the longest (2-byte stores into the transposed V cache): 3-4 % of the launch at 3072 to
    // 6552 rows; and for GELU on the widest tiles, one wave a SIMD, whose epilogue nothing else overlaps: 4096 x 8192 x 2048
    // 111.4 -> 109.7 us, 3280 x 7680 x 1920 102.9 -> 99.8, 16384 x 8192 x 2048 429 -> 416.  The others are short enough
    // that the hardware's own hand-over from a finished workgroup to the next does as well (+-2 %, GELU on 192x192 and
    // 224x192 +-1 %), so they keep one workgroup per tile.
    constexpr bool PERSIST = kPersistent<EPI, KG, SLICED, BM, BN>;
    const int n_tiles = p.tiles_m * p.tiles_n;
    int m0, n0;
#define FV_TILE_COORDS(vpid_)                                                                   \
    {                                                                                           \
        int pid_ = (vpid_);                                                                     \
        if ((n_tiles & 7) == 0) pid_ = (pid_ & 7) * (n_tiles >> 3) + (pid_ >> 3);              \
        constexpr int GROUP = 8;                                                                \
        const int per_group_ = GROUP * p.tiles_n;                                               \
        const int grp_ = pid_ / per_group_;                                                     \
        const int first_m_ = grp_ * GROUP;                                                      \
        const int gsize_ = min(p.tiles_m - first_m_, GROUP);                                    \
        const int in_grp_ = pid_ - grp_ * per_group_;                                           \
        m0 = (first_m_ + in_grp_ % gsize_) * BM;                                                \
        n0 = (in_grp_ / gsize_) * BN;                                                           \
    }
    int vpid = blockIdx.x;
    FV_TILE_COORDS(vpid)
    const int n_splits = SLICED ? p.splits : 1;
    const int split = SLICED ? (int)blockIdx.y : 0;
    const int KT = p.K / BK / n_splits;          // K tiles of this workgroup
    const bf16_t* const Ab = p.A + (size_t)split * KT * BK;
    const bf16_t* const Wb = p.W + (size_t)split * KT * BK;

    // Direct-to-LDS loads: one instruction moves 64 x 16 bytes into a contiguous
    // 1 KB of LDS (lane l lands at base + 16 l), i.e. RPI whole tile rows.  The
    // swizzle is applied on the global side: lane l fetches the chunk that
    // belongs at its LDS position.  Load j of a wave covers tile rows
    // (wave + NW j) * RPI + ld_row; the key of such a row does not depend on j
    // (RPI is 8 or 16, NW is even and the key uses row bits below 4).
    // Per-lane byte offsets of the loads; they do not change along K (the scalar
    // base pointer advances instead), so a load costs no vector arithmetic.
    uint32_t a_off[A_LD], w_off[W_LD];
#define FV_TILE_OFFSETS(lane_)                                                                  \
    {                                                                                           \
        const int ld_row_ = (lane_) / CPR;                                                      \
        const int ld_chunk_ = ((lane_) % CPR) ^ swz(wave * RPI + ld_row_);                 \
        _Pragma("unroll") for (int j = 0; j < A_LD; ++j)                                        \
            a_off[j] = (uint32_t)(min(m0 + (wave + NW * j) * RPI + ld_row_, p.M - 1) * p.K + ld_chunk_ * 8) * 2u; \
        _Pragma("unroll") for (int j = 0; j < W_LD; ++j)                                        \
            w_off[j] = (uint32_t)(min(n0 + (wave + NW * j) * RPI + ld_row_, p.N - 1) * p.K + ld_chunk_ * 8) * 2u; \
    }
    FV_TILE_OFFSETS(lane)

    typedef __attribute__((address_space(3))) void* lds_ptr_t;
#define FV_DMA16(base_, off_, lds_chunk_ptr_) load16_to_lds((base_), (off_), (uint32_t)(uintptr_t)(lds_ptr_t)(lds_chunk_ptr_))
    // Load q of a tile (A loads first, then W) into ring stage stage_.
#define FV_ISSUE_Q(kt_, stage_, q_)                                                             \
    {                                                                                           \
        if ((q_) < A_LD)                                                                        \
            FV_DMA16(Ab + (size_t)(kt_) * BK, a_off[(q_) < A_LD ? (q_) : 0],                   \
                     lds + (stage_) * STAGE + wave * 64 + (q_) * (NW * 64));                    \
        else                                                                                    \
            FV_DMA16(Wb + (size_t)(kt_) * BK, w_off[(q_) >= A_LD ? (q_) - A_LD : 0],           \
                     lds + (stage_) * STAGE + A_TILE + wave * 64 + ((q_) - A_LD) * (NW * 64));  \
    }
#define FV_ISSUE_TILE(kt_, stage_)                                                              \
    _Pragma("unroll") for (int q = 0; q < LPT; ++q) FV_ISSUE_Q(kt_, stage_, q)

    const int frag_row = lane & 15;
    const int frag_q = lane >> 4;
    const int a_row = wm * WTM + frag_row;  // + 16 mi
    const int w_row = wn * WTN + frag_row;  // + 16 ni
    const int frag_sw = swz(frag_row);

#define FV_LOAD_FRAGS(dst_a_, dst_w_, stage_, kk_)                                              \
    {                                                                                           \
        const u32x4_t* sa_ = lds + (stage_) * STAGE;                                            \
        const u32x4_t* sw_ = sa_ + A_TILE;                                                      \
        const int ch_ = (4 * (kk0 + (kk_)) + frag_q) ^ frag_sw;                              \
        _Pragma("unroll") for (int mi = 0; mi < MI; ++mi)                                       \
            dst_a_[mi] = *reinterpret_cast<const bf16x8_t*>(sa_ + (a_row + 16 * mi) * CPR + ch_); \
        _Pragma("unroll") for (int ni = 0; ni < NI; ++ni)                                       \
            dst_w_[ni] = *reinterpret_cast<const bf16x8_t*>(sw_ + (w_row + 16 * ni) * CPR + ch_); \
    }
    // The same operand reads with the loads of a whole tile issued between them, one after each read
    // (putting reads between the loads keeps the texture-address queue from filling up and stalling the wave).
    static_assert(kWide<BM, BN, WGM, WGN, KG> || LPT <= MI + NI, "a load for every operand read at most");
#define FV_LOAD_FRAGS_ISSUE(dst_a_, dst_w_, stage_, kk_, kt_, fill_)                            \
    {                                                                                           \
        const u32x4_t* sa_ = lds + (stage_) * STAGE;                                            \
        const u32x4_t* sw_ = sa_ + A_TILE;                                                      \
        const int ch_ = (4 * (kk0 + (kk_)) + frag_q) ^ frag_sw;                              \
        _Pragma("unroll") for (int g = 0; g < MI + NI; ++g) {                                   \
            if (g < MI)                                                                         \
                dst_a_[g < MI ? g : 0] =                                                        \
                    *reinterpret_cast<const bf16x8_t*>(sa_ + (a_row + 16 * g) * CPR + ch_);     \
            else                                                                                \
                dst_w_[g >= MI ? g - MI : 0] =                                                  \
                    *reinterpret_cast<const bf16x8_t*>(sw_ + (w_row + 16 * (g - MI)) * CPR + ch_); \
            if (g < LPT) FV_ISSUE_Q(kt_, fill_, g)                                              \
        }                                                                                       \
    }

    // Load q of K tile kt_ of either operand into stage stage_ of its ring (wide tiles).
#define FV_ISSUE_A(kt_, stage_, q_)                                                             \
    FV_DMA16(Ab + (size_t)(kt_) * BK, a_off[q_], lds + (stage_) * A_TILE + wave * 64 + (q_) * (NW * 64))
#define FV_ISSUE_W(kt_, stage_, q_)                                                             \
    FV_DMA16(Wb + (size_t)(kt_) * BK, w_off[q_], lds + SA * A_TILE + (stage_) * W_TILE + wave * 64 + (q_) * (NW * 64))

    // ---- prologue: AHEAD tiles in flight (EARLY: every stage of the ring)
    constexpr int AHEAD = EARLY ? STAGES : STAGES - 1;
    // wide tiles: what a hand-over's k-step still issues of the window that it opens (see the main loop)
    constexpr int SLOTS = MI * NI, SB = SLOTS >= 32 ? 4 : 2;             // slots of a k-step; those in front of the hand-over
    constexpr int RS = SLOTS - SB >= 2 * (MI + NI) ? 2 : 1;              // an operand read every RS slots
    constexpr int LS = WIDE ? load_slots(SLOTS, SB, KK, LPT) : 1;                 // a load every LS slots
    constexpr int W3 = handover_loads(SLOTS, SB, LS, LPT);
    static_assert(!WIDE || (LS > 0 && SLOTS - SB >= MI + NI && KK > 1), "a k-step has room for its reads, a K tile for its loads");
#define FV_ISSUE_PROLOGUE()                                                                     \
    if constexpr (WIDE) {                                                                       \
        static_for<0, STAGES - 1>([&](auto s_c) {                                               \
            constexpr int s = decltype(s_c)::value;                                             \
            if (s < KT) {                                                                       \
                if constexpr (s < SA - 1) {                                                     \
                    _Pragma("unroll") for (int q = 0; q < A_LD; ++q) FV_ISSUE_A(s, s, q);       \
                }                                                                               \
                _Pragma("unroll") for (int q = 0; q < W_LD; ++q) FV_ISSUE_W(s, s, q);           \
            }                                                                                   \
        });                                                                                     \
        if (SA - 1 < KT) {                                                                      \
            _Pragma("unroll") for (int q = 0; q < (W3 < A_LD ? W3 : A_LD); ++q) FV_ISSUE_A(SA - 1, SA - 1, q); \
        }                                                                                       \
        if (STAGES - 1 < KT) {                                                                  \
            _Pragma("unroll") for (int q = A_LD; q < W3; ++q) FV_ISSUE_W(STAGES - 1, STAGES - 1, q - A_LD < 0 ? 0 : q - A_LD); \
        }                                                                                       \
    } else {                                                                                    \
        _Pragma("unroll") for (int s = 0; s < AHEAD; ++s)                                       \
            if (s < KT) FV_ISSUE_TILE(s, s)                                                     \
    }
    // Rows of the residual and of the output, for the epilogue: asked for ahead of everything else, but where a wave has many of them
    // only behind the main loop, which needs the registers.
    constexpr bool RES = EPI == EPI_BIAS_RES && !SLICED, ROWS_EARLY = RES && MI <= 4;
    int res_row[RES ? MI : 1], out_row[RES ? MI : 1];
    auto load_rows = [&](int row) {
#pragma unroll
        for (int mi = 0; mi < (RES ? MI : 1); ++mi) res_row[mi] = out_row[mi] = min(m0 + wm * WTM + mi * 16 + row, p.M - 1);
        if (p.res_rows) {
#pragma unroll
            for (int mi = 0; mi < (RES ? MI : 1); ++mi) res_row[mi] = p.res_rows[res_row[mi]];
        }
        if (p.out_rows) {
#pragma unroll
            for (int mi = 0; mi < (RES ? MI : 1); ++mi) out_row[mi] = p.out_rows[out_row[mi]];
        }
    };
    if constexpr (ROWS_EARLY) load_rows(frag_row);
    FV_ISSUE_PROLOGUE()
    bool first_tile = true;
    for (;;) {   // the tiles of this workgroup
    // A lane's accumulators of 32 columns, in runs of four consecutive columns of one output row (see the epilogue).
    constexpr int RUNS = 2;
    auto run_col = [](int g, int q) { return 16 * g + 4 * q; };
    // The accumulators start from the bias, which saves the epilogue an add per element; with K split between
    // k-groups or workgroups only the first slice carries it.  (Accumulator blocks hold C transposed, see the
    // epilogue.)
    f32x4_t acc[MI][NI];
    u32x2_t bias[NJ][RUNS];
    const bool with_bias = p.bias && kg == 0 && split == 0;
#pragma unroll
    for (int i = 0; i < NJ * RUNS; ++i) bias[i / RUNS][i % RUNS] = u32x2_t{0u, 0u};
    if (with_bias) {   // (one branch, and addresses clamped instead of tested: all loads in flight at once)
#pragma unroll
        for (int i = 0; i < NJ * RUNS; ++i)
            bias[i / RUNS][i % RUNS] = *reinterpret_cast<const u32x2_t*>(
                p.bias + min(n0 + wn * WTN + (i / RUNS) * 32 + run_col(i % RUNS, frag_q), p.N - 4));
    }
#pragma unroll
    for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
        for (int g = 0; g < RUNS; ++g)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) {
                const u32x2_t bb = bias[nj][g];
                acc[mi][2 * nj + g] = f32x4_t{bf16_lo(bb.x), bf16_hi(bb.x), bf16_lo(bb.y), bf16_hi(bb.y)};
            }

    // ---- wait for the first K tile.  (A later tile of a persistent workgroup waits for everything: its
    // loads went out before the previous epilogue's stores and residual loads, and the counter says
    // nothing about the order in which loads and stores complete.)
    if (first_tile && KT >= (WIDE ? STAGES : AHEAD))
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(WIDE ? wide_out_at_start(SA, STAGES, A_LD, W_LD, W3) : (AHEAD - 1) * LPT, true));
    else
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    bf16x8_t fa[2][MI], fw[2][NI];
    if constexpr (WIDE) {
#define FV_WIDE_READ(set_, sa_, sw_, kk_, i_)                                                   \
    {                                                                                           \
        const int ch_ = (4 * (kk_) + frag_q) ^ frag_sw;                                     \
        if ((i_) == 0 || (i_) > NI)                                                             \
            fa[set_][(i_) > NI ? (i_) - NI : 0] = *reinterpret_cast<const bf16x8_t*>(           \
                lds + (sa_) * A_TILE + (a_row + 16 * ((i_) > NI ? (i_) - NI : 0)) * CPR + ch_); \
        else                                                                                    \
            fw[set_][(i_) > 0 && (i_) <= NI ? (i_) - 1 : 0] = *reinterpret_cast<const bf16x8_t*>( \
                lds + SA * A_TILE + (sw_) * W_TILE + (w_row + 16 * ((i_) > 0 ? (i_) - 1 : 0)) * CPR + ch_); \
    }
#pragma unroll
        for (int i = 0; i < MI + NI; ++i) FV_WIDE_READ(0, 0, 0, 0, i)
    } else {
        FV_LOAD_FRAGS(fa[0], fw[0], 0, 0)
    }

#define FV_MFMA_ROWS(cur_, mi_lo_, mi_hi_)                                                      \
    _Pragma("unroll") for (int mi = (mi_lo_); mi < (mi_hi_); ++mi)                              \
        _Pragma("unroll") for (int ni = 0; ni < NI; ++ni)                                       \
            acc[mi][ni] = mfma(fw[cur_][ni], fa[cur_][mi], acc[mi][ni]);
#define FV_INTERLEAVE(mfma_per_read_)                                                           \
    _Pragma("unroll") for (int g = 0; g < MI + NI; ++g) {                                       \
        __builtin_amdgcn_sched_group_barrier(0x008, (mfma_per_read_), 0); /* MFMA */            \
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                /* DS read */         \
    }
    // One K tile.  Software pipeline inside the wave: the operand reads of the
    // next k-step are interleaved with the MFMAs of the current one (the
    // scheduler is told the pattern), so LDS latency hides behind the matrix
    // pipe.  HANDOVER_: a next tile exists, so the last k-step waits for it (this
    // wave's loads: the counter, at most WAITN_ loads of later tiles still in
    // flight; the other waves' loads: the barrier, which also tells everyone that
    // this tile's stage is no longer being read) and preloads its first operands.
    // MORE_: a further tile is fetched, AHEAD tiles on: into the stage this tile
    // leaves, at its hand-over (EARLY), or into the stage the tile before it left,
    // during its first k-step.  The body is branch free on purpose: the
    // accumulators must stay in one register class across the loop.
#define FV_TILE_BODY(MORE_, HANDOVER_, WAITN_)                                                  \
    {                                                                                           \
        int next_stage_ = stage + 1;                                                            \
        if (next_stage_ == STAGES) next_stage_ = 0;                                             \
        int fill_ = stage + STAGES - 1;                                                         \
        if (fill_ >= STAGES) fill_ -= STAGES;                                                   \
        _Pragma("unroll") for (int kk = 0; kk < KK; ++kk) {                                     \
            const int cur_ = kk & 1, nxt_ = cur_ ^ 1;                                           \
            if (kk + 1 < KK) {                                                                  \
                if ((MORE_) && !EARLY)                                                          \
                    FV_LOAD_FRAGS_ISSUE(fa[nxt_], fw[nxt_], stage, kk + 1, kt + AHEAD, fill_) \
                else                                                                            \
                    FV_LOAD_FRAGS(fa[nxt_], fw[nxt_], stage, kk + 1)                            \
                FV_MFMA_ROWS(cur_, 0, MI)                                                       \
                FV_INTERLEAVE((MI * NI) / (MI + NI))                                            \
            } else if (HANDOVER_) {                                                             \
                __builtin_amdgcn_s_waitcnt(waitcnt_imm((WAITN_), true));                        \
                asm volatile("" ::: "memory");                                                  \
                __builtin_amdgcn_s_barrier();                                                   \
                asm volatile("" ::: "memory");                                                  \
                if ((MORE_) && EARLY)                                                           \
                    FV_LOAD_FRAGS_ISSUE(fa[nxt_], fw[nxt_], next_stage_, 0, kt + AHEAD, stage)  \
                else                                                                            \
                    FV_LOAD_FRAGS(fa[nxt_], fw[nxt_], next_stage_, 0)                           \
                FV_MFMA_ROWS(cur_, 0, MI)                                                       \
                FV_INTERLEAVE((MI * NI) / (MI + NI))                                            \
            } else {                                                                            \
                FV_MFMA_ROWS(cur_, 0, MI)                                                       \
            }                                                                                   \
        }                                                                                       \
        stage = next_stage_;                                                                    \
        if (KK == 1 && (HANDOVER_)) {   /* one k-step a tile: the next one's operands are in the other set */ \
            _Pragma("unroll") for (int mi = 0; mi < MI; ++mi) fa[0][mi] = fa[1][mi];            \
            _Pragma("unroll") for (int ni = 0; ni < NI; ++ni) fw[0][ni] = fw[1][ni];            \
        }                                                                                       \
    }

    if constexpr (WIDE) {
        // A slot is a matrix instruction and behind it at most one operand read, of the next k-step, and one load to LDS, fenced
        // off from the next slot.  The hand-over to the next K tile comes SB slots into the last k-step: this wave's loads of
        // that tile have landed (the counter), everyone's have, and nobody reads this tile's stages any more (the barrier).  It
        // opens the window in which the stages are refilled: the A tile SA on, then the W tile STAGES on, a load every LS slots,
        // through the rest of this k-step and the first ones of the next tile.  Three stages of W: weights come from memory,
        // rows from a cache.
        int sa = 0, sw = 0, kt = 0;
        auto body = [&](auto r_c) __attribute__((always_inline)) {
            constexpr int R = decltype(r_c)::value;      // tiles left after this one (at least)
            const int sa1 = sa + 1 == SA ? 0 : sa + 1, sw1 = sw + 1 == STAGES ? 0 : sw + 1;
            const int sap = sa == 0 ? SA - 1 : sa - 1, swp = sw == 0 ? STAGES - 1 : sw - 1;   // stages that the tile before left
            static_for<0, KK * SLOTS>([&](auto i_c) __attribute__((always_inline)) {
                constexpr int kk = decltype(i_c)::value / SLOTS, s = decltype(i_c)::value % SLOTS;
                constexpr int mi = s / NI, ni = s % NI, cur = kk & 1, nxt = cur ^ 1;
                constexpr bool last = kk == KK - 1;
                if constexpr (last && s == SB && R >= 1) {
                    __builtin_amdgcn_s_waitcnt(waitcnt_imm(wide_out_at_handover(SA, STAGES, A_LD, W_LD, R), true));
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                acc[mi][ni] = mfma(fw[cur][ni], fa[cur][mi], acc[mi][ni]);
                constexpr int rd = last ? (s >= SB && (s - SB) % RS == 0 ? (s - SB) / RS : -1) : (s % RS == 0 ? s / RS : -1);
                if constexpr (rd >= 0 && rd < MI + NI) {
                    if constexpr (!last) FV_WIDE_READ(nxt, sa, sw, kk + 1, rd)
                    else if constexpr (R >= 1) FV_WIDE_READ(nxt, sa1, sw1, 0, rd)
                }
                // loads: a window opens at a hand-over, for the stages that it frees; one every LS slots
                constexpr int q = last ? (s >= SB && (s - SB) % LS == 0 ? (s - SB) / LS : -1)
                                       : ((kk * SLOTS + s) % LS == LS / 2 ? W3 + (kk * SLOTS + s) / LS : -1);
                if constexpr (q >= 0 && q < A_LD) {
                    if constexpr (last && R >= SA) FV_ISSUE_A(kt + SA, sa, q);
                    if constexpr (!last && R >= SA - 1) FV_ISSUE_A(kt + SA - 1, sap, q);
                } else if constexpr (q >= A_LD && q < LPT) {
                    if constexpr (last && R >= STAGES) FV_ISSUE_W(kt + STAGES, sw, q - A_LD);
                    if constexpr (!last && R >= STAGES - 1) FV_ISSUE_W(kt + STAGES - 1, swp, q - A_LD);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            sa = sa1;
            sw = sw1;
            ++kt;
        };
        while (kt + STAGES < KT) body(std::integral_constant<int, STAGES>{});
        static_for<0, STAGES>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int r = STAGES - 1 - decltype(i_c)::value;
            if (KT - 1 - kt == r) body(std::integral_constant<int, r>{});
        });
    } else {
    int stage = 0;  // stage of tile kt
    int kt = 0;
    for (; kt + AHEAD < KT; ++kt) FV_TILE_BODY(true, true, (STAGES - 2) * LPT)
    // the ring drains: r tiles are left after this one, r-1 of them may still be in flight at the hand-over
    static_for<0, AHEAD - 1>([&](auto i_c) {
        constexpr int r = AHEAD - 1 - decltype(i_c)::value;
        if (KT - 1 - kt == r) {
            FV_TILE_BODY(false, true, (r - 1) * LPT)
            ++kt;
        }
    });
    FV_TILE_BODY(false, false, 0)
    }

    // This lane's place again, asked of the hardware: kept across the main loop it would cost the wide tiles a spill.
    const int lane_e = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int row_e = lane_e & 15, q_e = lane_e >> 4;

    // ---- the seam of a persistent workgroup: once every wave has read its last operands, the next tile's
    // first stages are fetched; the epilogue of this tile (m0e, n0e) runs under their flight
    const int m0e = m0, n0e = n0;
    const int vnext = vpid + (int)gridDim.x;
    const bool has_next = PERSIST && vnext < n_tiles;
    if (has_next) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(63, true));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        FV_TILE_COORDS(vnext)
        FV_TILE_OFFSETS(lane_e)
        FV_ISSUE_PROLOGUE()
    }

    // ---- Epilogue, from registers.  The MFMAs take the W fragment as their first operand, so an accumulator
    // block holds C transposed: register r of lane l is C[row, col] with row = l % 16 and col = 4*(l/16) + r inside a
    // 16x16 block: a lane owns one output row and a run of four consecutive columns, two runs in a pair of blocks.
    // GELU, residual and rotary turn are applied in fp32 per run, the runs are rounded once to bf16, and an exchange between
    // the quarters of the wave (v_permlane16_swap) leaves every lane with eight consecutive columns: a 16-byte store per
    // pair of blocks, no staging through LDS and no barrier between the main loop and the stores (a wave that is done
    // stores while the others still multiply).  The V section of the QKV GEMM is stored along the token axis of the transposed
    // cache: there consecutive lanes are consecutive tokens, 2-byte stores that a quarter of a wave makes 32 contiguous bytes.
    constexpr int XCH = KG > 1 ? MI * NI * 4 * 64 * NWQ : 0;  // floats handed over by the other k-groups
    static_assert(XCH * 4 <= STAGES * (BM + BN) * BK * 2, "the k-group exchange must fit in the tile LDS");
    if (KG > 1) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
        __builtin_amdgcn_s_barrier();  // every wave is done reading operand tiles: LDS is free for the exchange
        asm volatile("" ::: "memory");
    }
    if (KG > 1) {
        // Sum the k-groups: group g > 0 writes its accumulators (register-major, lane
        // contiguous), group 0 adds them; only group 0 goes on to the epilogue.
        float* xch = reinterpret_cast<float*>(smem) + wq * (MI * NI * 4 * 64) + lane_e;
        for (int g = 1; g < KG; ++g) {
            if (kg == g) {
                static_for<0, MI * NI * 4>([&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    xch[i * 64] = acc[i / (NI * 4)][(i / 4) % NI][i % 4];
                });
            }
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kg == 0) {
                static_for<0, MI * NI * 4>([&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    acc[i / (NI * 4)][(i / 4) % NI][i % 4] += xch[i * 64];
                });
            }
            if (g + 1 < KG) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, true));
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
        }
        if (kg != 0) return;  // no barrier follows
    }
    if constexpr (SLICED) {
        float* const sums = p.slices + (size_t)split * p.M * p.N;
        static_for<0, MI>([&](auto mi_c) {
            constexpr int mi = decltype(mi_c)::value;
            const int m = m0e + wm * WTM + mi * 16 + row_e;
            static_for<0, NJ * RUNS>([&](auto r_c) {
                constexpr int nj = decltype(r_c)::value / RUNS, g = decltype(r_c)::value % RUNS;
                const int n = n0e + wn * WTN + nj * 32 + run_col(g, q_e);
                if (m < p.M && n < p.N) *reinterpret_cast<f32x4_t*>(sums + (size_t)m * p.N + n) = acc[mi][2 * nj + g];
            });
        });
        return;
    }
    // The residual's loads go out RES_AHEAD row blocks ahead of their use, as many as fit into 64 registers, without a branch (columns
    // are clamped): loaded where they are added, each in a branch, a wave waited for memory once a run, and the epilogue of
    // out-proj and FC2 took half as long again.
    constexpr int RES_AHEAD = MI * NJ * RUNS * 2 <= 64 ? MI : 1;
    u32x2_t res[RES ? MI : 1][NJ * RUNS];
    auto load_residual = [&](auto mi_c) {
        constexpr int mi = decltype(mi_c)::value;
        const bf16_t* const row = p.residual + (size_t)res_row[RES ? mi : 0] * p.N;
#pragma unroll
        for (int i = 0; i < NJ * RUNS; ++i)
            res[RES ? mi : 0][i] = *reinterpret_cast<const u32x2_t*>(
                row + min(n0e + wn * WTN + (i / RUNS) * 32 + run_col(i % RUNS, q_e), p.N - 4));
    };
    if constexpr (RES && !ROWS_EARLY) load_rows(row_e);
    if constexpr (RES) static_for<0, RES_AHEAD>(load_residual);
    // Rotary positions, wide tiles: the slots of the wave's rows are fetched together, then a row block's angles together, one row block ahead,
    // both where registers are left, and without a branch (of columns past the keys any angle will do, it is not used).  Fetched where a run is turned,
    // the one wave of a SIMD waited for memory once a run: over the plain epilogue a round of 256x256 tiles took 19 us, now 10, of 192x192 10 and
    // 6, of 160x128 4.3 and 3.4 (QKV of 2048 / 4096 rows 2048 wide 56.5 -> 52.8, 110 -> 103, 3411 of 1536 64.0 -> 56.9, 7650 of 1024 74.4 -> 67.9).  Two waves
    // a SIMD cover each other, and lose 0.3 to 1 us a round by fetching more than they use.
    constexpr bool ROPE = EPI == EPI_QKV_ROPE, TURNS_EARLY = ROPE && WIDE;
    constexpr int TURN_AHEAD = MI * NI <= 48 ? 1 : 0, TURNS = TURNS_EARLY ? TURN_AHEAD + 1 : 1;
    constexpr bool SLOTS_EARLY = TURNS_EARLY && MI * NI <= 56;
    int slots[SLOTS_EARLY ? MI : 1];
    f32x2_t turn_cos[TURNS][NJ * RUNS], turn_sin[TURNS][NJ * RUNS];
    const bool turns = TURNS_EARLY && n0e + wn * WTN < 2 * p.D;   // (wave uniform: some of its columns are queries or keys)
    auto load_turn = [&](auto mi_c) {
        constexpr int mi = decltype(mi_c)::value;
        int slot = slots[SLOTS_EARLY ? mi : 0];
        if constexpr (!SLOTS_EARLY) {
            slot = min(m0e + wm * WTM + mi * 16 + row_e, p.M - 1);
            slot = p.rope_rows ? p.rope_rows[slot] % p.rope_N : slot % p.k_tokens;
        }
        const size_t lane_at = (size_t)slot * (p.dh >> 1) + 2 * q_e;
#pragma unroll
        for (int i = 0; i < NJ * RUNS; ++i) {
            const int first = ((n0e + wn * WTN + (i / RUNS) * 32) % p.dh + run_col(i % RUNS, 0)) / 2;
            turn_cos[mi % TURNS][i] = *reinterpret_cast<const f32x2_t*>(p.rope_cos + lane_at + first);
            turn_sin[mi % TURNS][i] = *reinterpret_cast<const f32x2_t*>(p.rope_sin + lane_at + first);
        }
    };
    if constexpr (SLOTS_EARLY) {
        if (turns) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) slots[mi] = min(m0e + wm * WTM + mi * 16 + row_e, p.M - 1);
            if (p.rope_rows) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi) slots[mi] = p.rope_rows[slots[mi]];
            }
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) slots[mi] = p.rope_rows ? slots[mi] % p.rope_N : slots[mi] % p.k_tokens;
            if constexpr (TURN_AHEAD > 0) load_turn(std::integral_constant<int, 0>{});
        }
    }
    static_for<0, MI>([&](auto mi_c) {
        constexpr int mi = decltype(mi_c)::value;
        const int m = m0e + wm * WTM + mi * 16 + row_e;
        const bool row_ok = m < p.M;
        const int mc = row_ok ? m : p.M - 1;
        // (sample, token) of this lane's row, where its output goes and where its residual comes from
        int bq = 0, tq = mc;
        if (is_qkv(EPI)) {
            bq = mc / p.k_tokens;
            tq = mc - bq * p.k_tokens;
        }
        const size_t orow = RES ? (size_t)out_row[RES ? mi : 0] : (size_t)mc;
        if constexpr (RES && mi + RES_AHEAD < MI) load_residual(std::integral_constant<int, mi + RES_AHEAD>{});
        bf16_t* const v_lane = p.v_cache + ((size_t)bq * p.H * p.dh + 4 * q_e) * p.L_cap + p.L0 + tq;
        if constexpr (TURNS_EARLY && mi + TURN_AHEAD < MI) {
            if (turns) load_turn(std::integral_constant<int, mi + TURN_AHEAD>{});
        }
        int slot = tq;   // the token's slot in its map
        if (ROPE && !TURNS_EARLY && p.rope_rows) slot = p.rope_rows[mc] % p.rope_N;
        static_for<0, NJ>([&](auto nj_c) {
            constexpr int nj = decltype(nj_c)::value;
            const int nb = n0e + wn * WTN + nj * 32;      // first column of the block (wave uniform)
            if (nb >= p.N) return;                       // N % 32 may be non-zero only past whole 8-column groups: checked per group below
            // QKV: section, head and channel of the block's first column (wave uniform: scalar arithmetic); the
            // 32 columns of a block lie in one section and one head (D and dh are multiples of 32)
            int sec = 0, f0 = 0, hh0 = 0, d0 = 0;
            if (is_qkv(EPI)) {
                sec = nb / p.D;
                f0 = nb - sec * p.D;
                hh0 = f0 / p.dh;
                d0 = f0 - hh0 * p.dh;
            }
            if (is_qkv(EPI) && sec == 2) {
                // V section: v_cache[b, head, d, L0 + t], consecutive lanes = consecutive tokens.  The address is a lane's
                // part, the same for all of a row's blocks, and a wave uniform one: per-lane column offsets were kept across
                // the rows, and spilled by the 256x256 tile
                if (row_ok) {
                    const size_t first = (size_t)hh0 * p.dh + d0;
                    static_for<0, RUNS * 4>([&](auto r_c) {
                        constexpr int r = decltype(r_c)::value, g = r >> 2;
                        v_lane[(first + 16 * g + (r & 3)) * p.L_cap] = (bf16_t)f32_to_bf16_bits(acc[mi][2 * nj + g][r & 3]);
                    });
                }
                return;
            }
            // two runs of four columns -> packed bf16 pairs
            uint32_t pk[RUNS][2];
            static_for<0, RUNS>([&](auto g_c) {
                constexpr int g = decltype(g_c)::value;
                const f32x4_t& c = acc[mi][2 * nj + g];
                float v[4] = {c[0], c[1], c[2], c[3]};
                if (EPI == EPI_BIAS_GELU) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = gelu_fast(v[j]);
                }
                if constexpr (RES) {
                    const u32x2_t rr = res[mi][nj * RUNS + g];
                    v[0] += bf16_lo(rr.x); v[1] += bf16_hi(rr.x);
                    v[2] += bf16_lo(rr.y); v[3] += bf16_hi(rr.y);
                }
                if constexpr (ROPE) {
                    // two interleaved pairs of one head, turned by the angles of the token's slot
                    f32x2_t cs = turn_cos[mi % TURNS][nj * RUNS + g], sn = turn_sin[mi % TURNS][nj * RUNS + g];
                    if constexpr (!TURNS_EARLY) {
                        const size_t at = (size_t)slot * (p.dh >> 1) + ((d0 + run_col(g, q_e)) >> 1);
                        cs = *reinterpret_cast<const f32x2_t*>(p.rope_cos + at);
                        sn = *reinterpret_cast<const f32x2_t*>(p.rope_sin + at);
                    }
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float a = v[2 * j], b = v[2 * j + 1];
                        v[2 * j] = a * cs[j] - b * sn[j];
                        v[2 * j + 1] = a * sn[j] + b * cs[j];
                    }
                }
                pk[g][0] = pack_bf16x2(v[0], v[1]);
                pk[g][1] = pack_bf16x2(v[2], v[3]);
            });
            // exchange between the quarters of the wave: the first and third give their second run and take the next quarter's
            // first one, so that a lane holds eight consecutive columns: 0-7, 16-23, 8-15 and 24-31 in quarter order
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const auto sw = __builtin_amdgcn_permlane16_swap(pk[0][c], pk[1][c], false, false);
                pk[0][c] = sw[0];
                pk[1][c] = sw[1];
            }
            {
                const int off = 16 * (q_e & 1) + 8 * (q_e >> 1);
                const int n8 = nb + off;      // first of this lane's eight columns
                if (row_ok && n8 < p.N) {
                    const u32x4_t o = {pk[0][0], pk[0][1], pk[1][0], pk[1][1]};
                    bf16_t* dst;
                    if (is_qkv(EPI)) {
                        if (sec == 0)   // q_out [B*k, D]
                            dst = p.q_out + ((size_t)bq * p.k_tokens + tq) * p.D + f0 + off;
                        else            // k_cache [B, H, L_cap, dh]
                            dst = p.k_cache + (((size_t)bq * p.H + hh0) * p.L_cap + p.L0 + tq) * p.dh + d0 + off;
                    } else {
                        dst = p.out + orow * p.N + n8;
                    }
                    *reinterpret_cast<u32x4_t*>(dst) = o;
                }
            }
        });
    });
    if (!has_next) break;
    vpid = vnext;
    first_tile = false;
    }   // the tiles of this workgroup
#undef FV_TILE_BODY
#undef FV_INTERLEAVE
#undef FV_MFMA_ROWS
#undef FV_ISSUE_PROLOGUE
#undef FV_ISSUE_TILE
#undef FV_ISSUE_Q
#undef FV_DMA16
#undef FV_LOAD_FRAGS_ISSUE
#undef FV_LOAD_FRAGS
#undef FV_TILE_OFFSETS
#undef FV_TILE_COORDS
#endif
}

// Compute units of the current device (asked once per process and device).
inline int compute_units() {
    static std::mutex mu;
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    std::lock_guard<std::mutex> lock(mu);
    if (cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cus[dev] = n;
    }
    return cus[dev];
}

template <int BM, int BN, int BK, int STAGES, int WGM, int WGN, int KG, int EPI, bool SLICED = false>
void launch_cfg(GemmParams& p, hipStream_t stream) {
    constexpr size_t smem = (kWide<BM, BN, WGM, WGN, KG> ? (size_t)kStagesA<BM, BN, BK, STAGES> * BM + (size_t)STAGES * BN
                                                         : (size_t)STAGES * (BM + BN)) * BK * sizeof(bf16_t);
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    static std::once_flag once;  // raising the dynamic-LDS limit is per function, once per process
    raise_lds_limit_once(once, &gemm_nt_kernel<BM, BN, BK, STAGES, WGM, WGN, KG, EPI, SLICED>, smem);
    if (!SLICED) p.splits = 1;
    // one round of workgroups when there are more tiles than the chip holds at a time (the kernel then walks
    // the rest itself); as many workgroups per CU as fit into its 160 KB of LDS
    int grid = p.tiles_m * p.tiles_n;
    if (kPersistent<EPI, KG, SLICED, BM, BN>) {
        constexpr int per_cu = (int)((160u << 10) / smem) > 0 ? (int)((160u << 10) / smem) : 1;
        const int slots = compute_units() * per_cu;
        if (grid > slots && slots % 8 == 0) grid = slots;
    }
    gemm_nt_kernel<BM, BN, BK, STAGES, WGM, WGN, KG, EPI, SLICED>
        <<<dim3(grid, SLICED ? p.splits : 1), 64 * WGM * WGN * KG, smem, stream>>>(p);
}

template <int EPI>
void launch_epi(GemmParams& p, hipStream_t stream) {
    int cfg = gemm_choose_tile(is_qkv(EPI), p.M, p.N, p.K).cfg;
    constexpr int knob = EPI == EPI_QKV_ROPE ? (int)EPI_QKV : EPI;
    if (gemm_cfg_override(knob) >= 0) cfg = gemm_cfg_override(knob);
    switch (cfg) {
        case TILE_256x256: launch_cfg<256, 256, 64, 3, 2, 2, 1, EPI>(p, stream); break;
        case TILE_256x192: launch_cfg<256, 192, 64, 3, 2, 2, 1, EPI>(p, stream); break;
        case TILE_224x256: launch_cfg<224, 256, 64, 3, 2, 2, 1, EPI>(p, stream); break;
        case TILE_224x192: launch_cfg<224, 192, 64, 3, 2, 2, 1, EPI>(p, stream); break;
        case TILE_224x128: launch_cfg<224, 128, 64, 3, 2, 2, 1, EPI>(p, stream); break;
        case TILE_192x256: launch_cfg<192, 256, 64, 3, 2, 2, 1, EPI>(p, stream); break;
        case TILE_192x192: launch_cfg<192, 192, 64, 3, 2, 2, 1, EPI>(p, stream); break;
        case TILE_160x128: launch_cfg<160, 128, 64, 4, 2, 2, 1, EPI>(p, stream); break;
        case TILE_256x128: launch_cfg<256, 128, 64, 3, 4, 2, 1, EPI>(p, stream); break;
        case TILE_192x128: launch_cfg<192, 128, 64, 3, 2, 4, 1, EPI>(p, stream); break;
        case TILE_128x64: launch_cfg<128, 64, 64, 6, 4, 2, 1, EPI>(p, stream); break;
        case TILE_64x64: launch_cfg<64, 64, 64, 4, 2, 2, 1, EPI>(p, stream); break;
        case TILE_64x64_DEEP:
            if constexpr (is_qkv(EPI)) {
                launch_cfg<64, 64, 64, 8, 2, 2, 1, EPI>(p, stream);
                break;
            }
            [[fallthrough]];
        case TILE_64x32: launch_cfg<64, 32, 64, 8, 2, 1, 2, EPI>(p, stream); break;
        default: launch_cfg<128, 128, 64, 4, 2, 4, 1, EPI>(p, stream); break;   // TILE_128x128
    }
}

}  // namespace

}  // namespace fv
