// Shared device-side helpers for the gfx950 kernels: bf16 pack/unpack, wave64
// reductions, vector types for MFMA operands.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace fv {

constexpr int kWave = 64;

typedef uint16_t bf16_t;  // raw bf16 bit pattern

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// bf16 -> fp32 is an exact widening: the 16 bits become the high half.
__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xFFFF0000u); }
__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// fp32 -> bf16, round to nearest even (NaN stays NaN): the hardware conversion
// of gfx950 (v_cvt_pk_bf16_f32), reached through the compiler's __bf16 type.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const f32x2_t f = {lo, hi};
    const bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
    return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) { return pack_bf16x2(f, 0.f) & 0xFFFFu; }

// Butterfly reductions over the 64 lanes of a wave; every lane gets the result
// and the combination order is fixed, so results are reproducible.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Eight bf16 values of a 16-byte vector, widened.
template <class V>
__device__ __forceinline__ void unpack8(const V& v, float (&f)[8]) {
    f[0] = bf16_lo(v.x); f[1] = bf16_hi(v.x);
    f[2] = bf16_lo(v.y); f[3] = bf16_hi(v.y);
    f[4] = bf16_lo(v.z); f[5] = bf16_hi(v.z);
    f[6] = bf16_lo(v.w); f[7] = bf16_hi(v.w);
}

// GELU in its tanh form written as a sigmoid: v * sigma(2u), u = sqrt(2/pi) (v + 0.044715 v^3).
// It deviates from the erf form by at most 3e-4 in absolute value (near |v| = 2),
// far below the bf16 resolution of the outputs, and costs 7 instructions where
// an erf approximation costs about 20: the epilogue is pure VALU time that no
// MFMA overlaps.
__device__ __forceinline__ float gelu_fast(float v) {
    // -2u log2(e), the factor folded into the two coefficients
    constexpr float c1 = -1.4426950408889634f * 1.5957691216057308f;
    constexpr float c3 = c1 * 0.044715f;
    const float v2 = v * v;
    const float e = __builtin_amdgcn_exp2f(v * fmaf(c3, v2, c1));                         // exp(-2u)
    return v * __builtin_amdgcn_rcpf(1.0f + e);
}

// LayerNorm of one row of D <= 512*CH columns by a wave, wherever one is computed: lane l holds the octets at columns
// 512 g + 8 l, statistics are two passes in fp32.  gain(g) and shift(g) give the lane's octet of either, store(g, v) takes
// the rounded result.
template <int CH, class Gain, class Shift, class Store>
__device__ __forceinline__ void layernorm_values(const uint4 (&raw)[CH], int D, float eps, Gain&& gain, Shift&& shift,
                                                 Store&& store) {
    const int lane = threadIdx.x & 63;
    float v[CH][8];
    float sum = 0.f;
#pragma unroll
    for (int g = 0; g < CH; ++g) {
        const int col = g * 512 + lane * 8;
        if (col < D) {
            unpack8(raw[g], v[g]);
#pragma unroll
            for (int j = 0; j < 8; ++j) sum += v[g][j];
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[g][j] = 0.f;
        }
    }
    const float mean = wave_sum(sum) / (float)D;
    float sq = 0.f;
#pragma unroll
    for (int g = 0; g < CH; ++g) {
        const int col = g * 512 + lane * 8;
        if (col < D) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float d = v[g][j] - mean;
                sq = fmaf(d, d, sq);
            }
        }
    }
    const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)D + eps);
#pragma unroll
    for (int g = 0; g < CH; ++g) {
        const int col = g * 512 + lane * 8;
        if (col < D) {
            float gm[8], bt[8];
            unpack8(gain(g), gm);
            unpack8(shift(g), bt);
            float o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = fmaf((v[g][j] - mean) * rstd, gm[j], bt[j]);
            uint4 pk;
            pk.x = pack_bf16x2(o[0], o[1]);
            pk.y = pack_bf16x2(o[2], o[3]);
            pk.z = pack_bf16x2(o[4], o[5]);
            pk.w = pack_bf16x2(o[6], o[7]);
            store(g, pk);
        }
    }
}

// 64 x 16 bytes from base + a lane's byte offset into 1 KB of LDS (lane l at lds + 16 l), through inline assembly: the compiler's own
// model of this instruction makes it drain every outstanding LDS operation before the next operand use, which would
// serialise the operand reads behind it.  Completion is tracked by hand (vmcnt before the barrier that publishes a tile).
__device__ __forceinline__ void load16_to_lds(const void* base, uint32_t offset, uint32_t lds) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(offset), "s"(base) : "memory", "m0");
#endif
}

// Compile-time loop: f(integral_constant<int, I>) for I in [Begin, End).
// Used where an accumulator array must only ever be indexed by constants.
template <int Begin, int End, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (Begin < End) {
        f(std::integral_constant<int, Begin>{});
        static_for<Begin + 1, End>(f);
    }
}

}  // namespace fv
