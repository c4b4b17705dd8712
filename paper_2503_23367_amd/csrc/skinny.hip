// GEMMs of at most kFewRowsMax rows (the first scales of a schedule): C[m,n] = sum_k A[m,k] * W[n,k], with the
// same fused epilogues as gemm_tiles.h and, for the QKV and FC1 products, the LayerNorm of the rows in front.
//
// At these row counts a block is one pass over its weights (100 MB for the large model), and the time goes to what
// surrounds that pass: a launch per LayerNorm, rings that fill and drain, partial tiles that travel through
// memory between workgroups.  So no weights are staged here: a workgroup owns CW output columns over the whole K
// range, its waves take K in turns of 64, and every lane loads its weights straight from memory into the
// registers of a 16x16x32 MFMA operand, all loads of a wave in flight at once (a weight is used by one wave
// only, so LDS would add a trip and save nothing).  The waves' sums meet in LDS, in wave order; nothing is
// exchanged between workgroups.
//
// LN: the rows are loaded first and the weights right behind them; the rows are normalised, a wave a row, while the
// weights are on their way, and reach the operands through LDS.  Every workgroup repeats this for its columns: 16 rows
// from L2.  (Every wave normalising its own share of all sixteen operand rows, also those beyond M: eight blocks of one
// token 357 us, this way 326.)
//
// Eight blocks of the large model (805 MB of weights), against the tiled products: one row 465 -> 335 us, 16 rows 472 -> 411;
// of the 512 px model 481 -> 301, 494 -> 392; of the small model 308 -> 185, 319 -> 245.  Beyond 16 rows it loses (25 rows in two
// groups 660 against 474 us: every workgroup reads the rows' operands from L2, and they no longer fit beside the
// weights in registers), hence kFewRowsMax; launch_math.h says which shapes of up to 16 rows come here.
//
// CW = 16 fills the operand with 16 weight rows; 12 leaves a quarter of it to repetitions of the last one, for the sake of how many
// workgroups there are (few_rows_columns).  CW = 8 (outputs of few columns: out-proj, FC2) gives half of the
// operand's rows to a second K half of the same eight columns, which doubles the number of workgroups: the matrix
// instructions, one per half, waste half of their rows, and have the time.
#include "common.h"
#include "kernels.h"
#include "launch_math.h"

namespace fv {

namespace {

__device__ __forceinline__ u32x4_t load16(const void* p) { return *reinterpret_cast<const u32x4_t*>(p); }

__device__ __forceinline__ f32x4_t mfma16(const u32x4_t& w, const u32x4_t& a, const f32x4_t& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, a), c,
                                                   0, 0, 0);
}

// A barrier for what is in LDS: __syncthreads() would wait for the weights in flight as well.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Lane l of a wave: operand row r = l % 16 (weight row n0 + r, or token row r of a 16-row group) and K octets
// q = l / 16 of a 64-wide turn: elements [16 q, 16 q + 16) in two 16-byte loads, one per MFMA (K may be taken in any
// order as long as both operands agree; this one makes a turn's two loads of a row one 128-byte line).
// U: turns a wave has in flight.  Turns past the end load the last one and are skipped by a wave-uniform branch around
// the MFMA, not around the load: with loads in branches the compiler can no longer count what is in flight, and waits for all.
// Results: lane l holds columns n0 + 4 q + 0..3 of token row r.
// ROWS (no LN): the rows' operands come from LDS, where the workgroup has laid all of the rows; without it every lane of a wave loads its
// own, sixteen rows' worth whatever M is, and a product of one row over K = 8192 spent more of its time on those than on its weights.
template <int EPI, bool LN, int CW, int NW, int U, bool ROWS = false>
__global__ __launch_bounds__(64 * NW) void skinny_kernel(const GemmArgs p) {
    constexpr int KH = CW == 8 ? 2 : 1;               // K halves side by side in the weight operand
    __shared__ f32x4_t red[NW][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 15, q = lane >> 4;
    const int n0 = blockIdx.x * CW;
    const int turns = p.K >> 6;
    const int half = (turns + KH - 1) / KH;           // turns of the first K half

    if (LN && blockIdx.x == 0) {                      // (the launch stands in for the call's first LayerNorm)
        for (int i = threadIdx.x; i < p.zero.n; i += 64 * NW) p.zero.p[i] = 0;
    }

    // this lane's weight row, and the turn its K half starts at
    const int wh = KH == 2 ? r >> 3 : 0;
    const bf16_t* const wrow = static_cast<const bf16_t*>(p.W) +
                               (size_t)min(n0 + (KH == 2 ? (r & 7) : min(r, CW - 1)), p.N - 1) * p.K + 16 * q;
    // (rows past M repeat the last one; their results are dropped)
    const bf16_t* const arow = static_cast<const bf16_t*>(p.A) + (size_t)min(r, p.M - 1) * p.K + 16 * q;

    // what the epilogue reads (this lane's four columns of row m) goes out ahead of everything else, without a branch
    const int m = r, mc = min(m, p.M - 1);
    const int n = n0 + 4 * q, nc = min(n, p.N - 4);
    const u32x2_t bias = *reinterpret_cast<const u32x2_t*>(static_cast<const bf16_t*>(p.bias ? p.bias : p.W) + nc);
    u32x2_t res = {0u, 0u};
    size_t orow = (size_t)mc;
    if (EPI == EPI_BIAS_RES) {
        const size_t rrow = p.res_rows ? (size_t)p.res_rows[mc] : (size_t)mc;
        if (p.out_rows) orow = (size_t)p.out_rows[mc];
        res = *reinterpret_cast<const u32x2_t*>(static_cast<const bf16_t*>(p.residual) + rrow * p.N + nc);
    }

    f32x4_t acc[KH];
#pragma unroll
    for (int h = 0; h < KH; ++h) acc[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    if constexpr (LN) {
        static_assert(!LN || (CW != 8 && 2 * 8 * NW * U <= 64 * NW), "one K range; gain and shift fit where the sums go");
        // The rows are normalised as a LayerNorm launch does it, by the same code: a wave has one or two of them, in
        // registers, and leaves them in LDS, where the waves find their operands (16 bytes of padding a row: the sixteen
        // rows of an operand in different banks).  So a row has the same bits here as with an index list, whose gather is
        // such a launch, and its arithmetic is done once a workgroup.  Gain and shift, the same for all rows, go through
        // LDS too: in registers they would cost a second workgroup per CU, and the QKV and FC1 grids of the large model
        // are one and a half to two workgroups per CU.
        extern __shared__ __attribute__((aligned(16))) bf16_t rows_s[];
        const int stride = p.K + 8;
        u32x4_t(*const gb)[8 * NW * U] = reinterpret_cast<u32x4_t(*)[8 * NW * U]>(&red[0][0]);
        const int octets = p.K >> 3;                  // 16-byte chunks of a row: at most 8 * NW * U
        uint4 raw[2][U];
        u32x4_t w[U][2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (wave + NW * h < p.M) {
                const bf16_t* const src = static_cast<const bf16_t*>(p.A) + (size_t)(wave + NW * h) * p.K;
#pragma unroll
                for (int g = 0; g < U; ++g)
                    raw[h][g] = *reinterpret_cast<const uint4*>(src + min(g * 512 + lane * 8, p.K - 8));
            }
        // thread t fetches chunk t of [gain | shift]
        const int t0 = threadIdx.x;
        const int chunk = min(t0 < octets ? t0 : t0 - octets, octets - 1);
        const u32x4_t gv = load16(static_cast<const bf16_t*>(t0 < octets ? p.ln_g : p.ln_b) + chunk * 8);
        __builtin_amdgcn_sched_barrier(0);            // loads complete in order: the weights go out last
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) w[i][c] = load16(wrow + min(wave + NW * i, turns - 1) * 64 + 8 * c);
        __builtin_amdgcn_sched_barrier(0);
        if (t0 < 2 * octets) gb[t0 < octets ? 0 : 1][chunk] = gv;
        lds_barrier();
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (wave + NW * h < p.M)
                layernorm_values<U>(raw[h], p.K, p.ln_eps, [&](int g) { return gb[0][g * 64 + lane]; },
                                    [&](int g) { return gb[1][g * 64 + lane]; },
                                    [&](int g, const uint4& v) {
                                        *reinterpret_cast<uint4*>(rows_s + (wave + NW * h) * stride + g * 512 + lane * 8) = v;
                                    });
        lds_barrier();
        const bf16_t* const xrow = rows_s + min(r, p.M - 1) * stride + 16 * q;
        u32x4_t a[U][2];
#pragma unroll
        for (int i = 0; i < U; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) a[i][c] = load16(xrow + min(wave + NW * i, turns - 1) * 64 + 8 * c);
#pragma unroll
        for (int i = 0; i < U; ++i)
            if (wave + NW * i < turns) {
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[0] = mfma16(w[i][c], a[i][c], acc[0]);
            }
    } else {
        extern __shared__ __attribute__((aligned(16))) u32x4_t chunks_s[];
        const int cpr = p.K >> 3;                     // 16-byte chunks of a row
        if constexpr (ROWS) {
            // straight into LDS, 64 chunks a load; chunk c of row m at c ^ (m % 8), so that an operand's rows are in different banks
            typedef __attribute__((address_space(3))) void* lds_ptr_t;
            const int total = p.M * cpr;
            for (int s0 = wave * 64; s0 < total; s0 += NW * 64) {
                const int s = min(s0 + lane, total - 1), row = s / cpr, c = s - row * cpr;
                load16_to_lds(p.A, (uint32_t)(row * cpr + (c ^ (row & 7))) * 16u, (uint32_t)(uintptr_t)(lds_ptr_t)(chunks_s + s0));
            }
        }
        const int am = min(r, p.M - 1);
        const u32x4_t* const achunk = chunks_s + am * cpr;
        auto round = [&](int base, bool first) __attribute__((always_inline)) {
            u32x4_t w[U][2], a[U][KH][2];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int t = min(base + wave + NW * i, half - 1);
#pragma unroll
                for (int c = 0; c < 2; ++c) w[i][c] = load16(wrow + min(t + wh * half, turns - 1) * 64 + 8 * c);
            }
            if (ROWS && first) {
                // loads return in order: all but the 2 U of the weights behind the rows
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * U) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int t = min(base + wave + NW * i, half - 1);
#pragma unroll
                for (int h = 0; h < KH; ++h)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int turn = min(t + h * half, turns - 1);
                        if constexpr (ROWS) a[i][h][c] = achunk[turn * 8 + ((2 * q + c) ^ (am & 7))];
                        else a[i][h][c] = load16(arow + turn * 64 + 8 * c);
                    }
            }
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int t = base + wave + NW * i;
#pragma unroll
                for (int h = 0; h < KH; ++h)
                    if (t < half && t + h * half < turns) {
#pragma unroll
                        for (int c = 0; c < 2; ++c) acc[h] = mfma16(w[i][c], a[i][h][c], acc[h]);
                    }
            }
        };
        round(0, true);
        for (int base = NW * U; base < half; base += NW * U) round(base, false);
    }

    if (KH == 2) {
        // columns 0-7 of the first half are in lanes 0-31 of its results, those of the second half in lanes
        // 32-63 of its own (each MFMA's other half multiplied mismatched K ranges and is dropped)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[0][j] += __shfl_xor(acc[KH - 1][j], 32, 64);
    }
    red[wave][lane] = acc[0];
    __syncthreads();
    if (wave != 0 || m >= p.M || 4 * q >= CW || n >= p.N) return;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (p.bias) { v[0] = bf16_lo(bias.x); v[1] = bf16_hi(bias.x); v[2] = bf16_lo(bias.y); v[3] = bf16_hi(bias.y); }
    f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < NW; ++x) sum += red[x][lane];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] += sum[j];

    if (EPI == EPI_BIAS_GELU) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = gelu_fast(v[j]);
    }
    if (EPI == EPI_BIAS_RES) {
        v[0] += bf16_lo(res.x); v[1] += bf16_hi(res.x);
        v[2] += bf16_lo(res.y); v[3] += bf16_hi(res.y);
    }
    bf16_t* dst;
    if (is_qkv(EPI)) {
        const int sec = n / p.D, f = n - sec * p.D, hh = f / p.dh, d = f - hh * p.dh;
        const int bq = m / p.k_tokens, tq = m - bq * p.k_tokens;
        if (sec == 2) {
            bf16_t* const vc =
                static_cast<bf16_t*>(p.v_cache) + (((size_t)bq * p.H + hh) * p.dh + d) * p.L_cap + p.L0 + tq;
#pragma unroll
            for (int j = 0; j < 4; ++j) vc[(size_t)j * p.L_cap] = (bf16_t)f32_to_bf16_bits(v[j]);
            return;
        }
        if (EPI == EPI_QKV_ROPE) {
            const int slot = p.rope_rows ? p.rope_rows[m] % p.rope_N : tq;
            const size_t at = (size_t)slot * (p.dh >> 1) + (d >> 1);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float cs = p.rope_cos[at + j], sn = p.rope_sin[at + j], x = v[2 * j], y = v[2 * j + 1];
                v[2 * j] = x * cs - y * sn;
                v[2 * j + 1] = x * sn + y * cs;
            }
        }
        if (sec == 0) dst = static_cast<bf16_t*>(p.q_out) + (size_t)m * p.D + f;
        else dst = static_cast<bf16_t*>(p.k_cache) + (((size_t)bq * p.H + hh) * p.L_cap + p.L0 + tq) * p.dh + d;
    } else {
        dst = static_cast<bf16_t*>(p.out) + orow * p.N + n;
    }
    *reinterpret_cast<u32x2_t*>(dst) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}

template <int EPI, bool LN, int CW, int NW, int U>
void launch(const GemmArgs& a, hipStream_t st) {
    const int grid = (a.N + CW - 1) / CW;
    if constexpr (LN) {   // sixteen rows of 2048 columns: 74 KB with the sums, two workgroups in a CU's 160 KB
        static std::once_flag once;
        raise_lds_limit_once(once, &skinny_kernel<EPI, LN, CW, NW, U>, kFewRowsMax * (512 * U + 8) * sizeof(bf16_t));
        skinny_kernel<EPI, LN, CW, NW, U><<<grid, 64 * NW, (size_t)a.M * (a.K + 8) * sizeof(bf16_t), st>>>(a);
    } else if (few_rows_in_lds(a.M, a.N, a.K, EPI != EPI_BIAS_RES)) {
        static std::once_flag once;
        raise_lds_limit_once(once, &skinny_kernel<EPI, LN, CW, NW, U, true>, kFewRowsLds);
        const size_t rows_bytes = ((size_t)a.M * a.K * sizeof(bf16_t) + 1023) / 1024 * 1024;   // whole loads
        skinny_kernel<EPI, LN, CW, NW, U, true><<<grid, 64 * NW, rows_bytes, st>>>(a);
    } else {
        skinny_kernel<EPI, LN, CW, NW, U><<<grid, 64 * NW, 0, st>>>(a);
    }
}

template <int EPI, bool LN, int CW, int NW, int U>
void launch_turns(int turns, const GemmArgs& a, hipStream_t st) {
    if constexpr (U > 1)
        if (turns < U) return launch_turns<EPI, LN, CW, NW, U - 1>(turns, a, st);
    launch<EPI, LN, CW, NW, U>(a, st);
}

template <int EPI>
void launch_epi(const GemmArgs& a, hipStream_t st) {
    constexpr int W = kFewRowsWaves, U = kFewRowsTurns;
    const FewRowsPlan p = few_rows_plan(a.N, a.K, EPI != EPI_BIAS_RES);
    if constexpr (EPI != EPI_BIAS_RES)
        if (a.ln_g) return few_rows_columns(a.N) == 12 ? launch_turns<EPI, true, 12, W, U>(p.turns, a, st)
                                                       : launch_turns<EPI, true, 16, W, U>(p.turns, a, st);
    if (p.cols == 16) launch_turns<EPI, false, 16, W, U>(p.turns, a, st);
    else if (p.waves == W) launch_turns<EPI, false, 8, W, U>(p.turns, a, st);
    else launch_turns<EPI, false, 8, 2 * W, U>(p.turns, a, st);
}

}  // namespace

void launch_gemm_skinny(GemmEpilogue epi, const GemmArgs& a, hipStream_t stream) {
    switch (epi) {
        case EPI_QKV:
            if (a.rope_cos) launch_epi<EPI_QKV_ROPE>(a, stream);
            else launch_epi<EPI_QKV>(a, stream);
            break;
        case EPI_BIAS_RES: launch_epi<EPI_BIAS_RES>(a, stream); break;
        case EPI_BIAS_GELU: launch_epi<EPI_BIAS_GELU>(a, stream); break;
    }
}

}  // namespace fv
