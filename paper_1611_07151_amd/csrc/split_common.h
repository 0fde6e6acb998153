// fp32 contractions on the f16 matrix instructions (internal).
//
// An fp32 value scaled by a power of two into the upper part of the f16 range is the sum of two f16 values, hi + lo,
// up to 2^-24 of itself (hi rounded to nearest leaves 12 bits and a sign, lo keeps 11 of them).  A product of two such
// sums is hi*hi + hi*lo + lo*hi; the dropped lo*lo is below 2^-24 of it.  So three v_mfma_f32_32x32x16_f16 with fp32
// accumulation do the work of eight v_mfma_f32_32x32x2_f32: 96 against 512 cycles of a SIMD's matrix unit.  Measured
// on uniform and normal operands, relative 2-norm error against 64-bit sums, this form / the fp32 instructions:
// 1.2e-7 / 1.2e-7 at 96 terms, 3.0e-7 / 3.3e-7 at 576, 5.3e-7 / 5.9e-7 at 2304 (one accumulator; with the two cross
// terms in an accumulator of their own, as here, the sum is rounded a third as often).
//
// Scales are powers of two, so applying and removing them is exact: kernels get one per output layer, activations one
// per pixel tile or pixel, chosen from the largest magnitude there.  f16 holds 2^-24 .. 2^15, so values down to 2^-17
// of the scale's reference keep all their bits and smaller ones an absolute error of 2^-40 of it.
#pragma once

#include "conv_mfma_common.h"

namespace sq {
namespace split {

using namespace mfma;

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));   // four floats at any fp32 address

// An infinity or NaN has no hi and lo: sums that it may reach are made from the fp32 operands instead.
__device__ __forceinline__ bool odd8(const float *v)
{
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) m = max(m, __builtin_bit_cast(uint32_t, v[k]) & 0x7fffffffu);
    return m >= 0x7f800000u;
}
constexpr int kPlainRow = 1 << 30;    // in the place of a scale's exponent: an output layer whose kernels hold such a value
// Magnitude bits of a finite value; infinities and NaN count as zero, so that they do not set a scale.
__device__ __forceinline__ uint32_t magnitude(float v)
{
    const uint32_t m = __builtin_bit_cast(uint32_t, v) & 0x7fffffffu;
    return m >= 0x7f800000u ? 0u : m;
}
// The largest magnitude of eight values (the exact rule for infinities and NaN only where one is there).
__device__ __forceinline__ uint32_t magnitude8(const float *v)
{
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) m = max(m, __builtin_bit_cast(uint32_t, v[k]) & 0x7fffffffu);
    if (__ballot(m >= 0x7f800000u)) {
        m = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) m = max(m, magnitude(v[k]));
    }
    return m;
}
// Exponent of the power of two that brings a magnitude (bits) into [2^13, 2^14), one factor of two of room below 2^15;
// 127 at most (zero and the smallest values).  Scales are kept as exponents: they are removed with ldexp, which neither
// over- nor underflows on the way where the product of two powers of two would.
__device__ __forceinline__ int scale_exponent(uint32_t mag) { return min(140 - (int)(mag >> 23), 127); }
__device__ __forceinline__ float pow2(int e) { return __builtin_bit_cast(float, (uint32_t)(e + 127) << 23); }   // -126 .. 127

// Largest / smallest of a wavefront's 64 lanes, the same in all: shifts within rows of 16, then row 0's and the first two
// rows' results passed on, by DPP (a lane that nothing is shifted into keeps its own value).
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
#define SQ_STEP(ctrl) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, 0xf, 0xf, false))
    SQ_STEP(0x111); SQ_STEP(0x112); SQ_STEP(0x114); SQ_STEP(0x118); SQ_STEP(0x142); SQ_STEP(0x143);
#undef SQ_STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) { return ~wave_max(~v); }

// Sum over a half wavefront's 32 lanes, in its last lane (31 and 63).
__device__ __forceinline__ float half_wave_sum(float v)
{
#define SQ_STEP(ctrl, rows) v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, rows, 0xf, false))
    SQ_STEP(0x111, 0xf); SQ_STEP(0x112, 0xf); SQ_STEP(0x114, 0xf); SQ_STEP(0x118, 0xf); SQ_STEP(0x142, 0xa);
#undef SQ_STEP
    return v;
}

// Two values as hi and lo pairs: one packed conversion, two subtractions that round to f16.
__device__ __forceinline__ void split2(float a, float b, uint32_t &hi, uint32_t &lo)
{
    asm volatile("" : "+v"(a), "+v"(b));     // (else the scaling is folded into three instructions per value instead of one)
    const f16x2 h = {(_Float16)a, (_Float16)b};
    const f16x2 l = {(_Float16)(a - (float)h.x), (_Float16)(b - (float)h.y)};
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}
__device__ __forceinline__ void split8(const float *v, float s, u32x4 &hi, u32x4 &lo)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint32_t h, l;
        split2(v[2 * k] * s, v[2 * k + 1] * s, h, l);
        hi[k] = h;
        lo[k] = l;
    }
}
__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

}  // namespace split
}  // namespace sq
