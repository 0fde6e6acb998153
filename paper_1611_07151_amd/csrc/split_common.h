// fp32 contractions on the f16 matrix instructions (internal).
//
// An fp32 value scaled by a power of two into the upper part of the f16 range is hi + lo / 2^11, both f16: hi rounded to
// nearest leaves a remainder of at most 2^-11 of the value's binade, of which lo keeps 11 bits.  Three quarters of all fp32
// values are held exactly, the others up to their last bit, 2^-23 of the value at most.  A product of two such sums is
// hi*hi + (hi*lo + lo*hi) / 2^11; the dropped lo*lo is at most 2^-22 of it, 2^-24 as a rule.  So three
// v_mfma_f32_32x32x16_f16 with fp32 accumulation, the cross terms in an accumulator of their own, do the work of eight
// v_mfma_f32_32x32x2_f32: 96 against 512 cycles of a SIMD's matrix unit.  What the operands lose is less than what the
// fp32 instructions lose in their longer chain of additions (16 terms are added per rounding instead of two).
//
// Scales are powers of two, so applying and removing them is exact: kernels get one per output layer, activations one
// per pixel tile or pixel, chosen from the largest magnitude there, which comes to lie in [2^13, 2^14).  lo ends at 2^-24,
// that is 2^-35 of hi's units: values from 2^-25 of the largest on keep all their bits, smaller ones are held to an
// absolute 2^-36 (2^-49 of the largest).  That is no loss to a sum that a larger term reaches, but it is where the larger
// ones meet zeros.  So tiles and output layers with a non-zero value below 2^-27 of their largest are marked (kWide; a value
// just above it still has 22 bits), and of their sums those that stay below kSmall (2^-22 of one large product and less: what
// the operands lose is then no longer far below what the sum's own roundings are) are made again on the fp32
// instructions, from memory, as are all that an infinity or NaN may reach.  Normally distributed values give a mark to
// one tile or layer in some thousands, and such a sum to one call in some thousands (with marks from 2^-25 and sums below
// 64 of all layers of a block: one call in twenty, 50 us each).
#pragma once

#include "conv_mfma_common.h"

namespace sq {
namespace split {

using namespace mfma;

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));   // four floats at any fp32 address

constexpr int kLowBits = 11;                       // lo is kept times 2^11
constexpr uint32_t kWide = 27u << 23;              // spread of magnitudes (as bits) from which a set is marked
constexpr float kSmall = 16.f;                     // sums of marked tiles and layers below this, scales included, are made again
// Range of the magnitudes of a set of values: the largest (NaN if one is), and the smallest but zero as twice its bits less
// one (~0 if there is none).  Two instructions per value.
struct Range {
    float top = 0.f;
    uint32_t low = ~0u;
    __device__ __forceinline__ void add2(float a, float b)
    {
        top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(top, fabsf(a)), fabsf(b));
        low = min(low, min((__builtin_bit_cast(uint32_t, a) << 1) - 1u, (__builtin_bit_cast(uint32_t, b) << 1) - 1u));
    }
    __device__ __forceinline__ void add8(const float *v)
    {
#pragma unroll
        for (int k = 0; k < 8; k += 2) add2(v[k], v[k + 1]);
    }
    __device__ __forceinline__ uint32_t top_bits() const { return __builtin_bit_cast(uint32_t, top) & 0x7fffffffu; }
};
constexpr uint32_t kOddMagnitude = 0x7f800000u;      // bits of an infinity; above: NaN
__device__ __forceinline__ bool spread(uint32_t top_bits, uint32_t low) { return top_bits > (low >> 1) && top_bits - (low >> 1) >= kWide; }
// An output layer's scale and marks in one word: the exponent in the lower 16 bits, and
constexpr int kWideRow = 1 << 16, kOddRow = 1 << 17;      // its kernels are spread wide / hold an infinity or NaN
__device__ __forceinline__ int row_exponent(int row) { return (int)(short)row; }
__device__ __forceinline__ int row_word(int exponent, uint32_t top, uint32_t low)
{
    return (exponent & 0xffff) | (spread(top, low) ? kWideRow : 0) | (top >= kOddMagnitude ? kOddRow : 0);
}
// Exponent of the power of two that brings a magnitude (bits) into [2^13, 2^14), one factor of two of room below 2^15;
// 127 at most (zero and the smallest values: their last bits lie above 2^-36 all the same).  Scales are kept as exponents: they are removed with ldexp, which neither
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

// Two values as hi and lo pairs.
__device__ __forceinline__ void split2(float a, float b, uint32_t &hi, uint32_t &lo)
{
    asm volatile("" : "+v"(a), "+v"(b));     // (else the scaling is folded into three instructions per value instead of one)
    constexpr float up = 1 << kLowBits;
    const f16x2 h = {(_Float16)a, (_Float16)b};
    const f16x2 l = {(_Float16)((a - (float)h.x) * up), (_Float16)((b - (float)h.y) * up)};
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
// Eight kernel values.  What a kernel loses is the same for every pixel, and an average over pixels does not take it away as
// it does an activation's.  A value that lo does not hold lies half-way between two that it does: of the two the one is
// taken that brings the sum of the errors so far (`off`) back towards zero.  Class means of the network at 64 images,
// relative error: fp32 instructions 1.17e-7, split with each value rounded by itself 1.45e-7, so 1.35e-7.  (Carried on over
// the taps of a kernel as well 1.35e-7, but 5 us more for a layer's kernels; in the 1x1 kernels that a wavefront splits
// on its way 1.32e-7, but 3 to 4 us more per launch.)
__device__ __forceinline__ void split8_kernel(const float *v, float s, u32x4 &hi, u32x4 &lo, float &off)
{
    constexpr float up = 1 << kLowBits;
    _Float16 h[8], l[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float a = v[k] * s;
        h[k] = (_Float16)a;
        const float rest = (a - (float)h[k]) * up;
        l[k] = (_Float16)rest;
        const float error = (float)l[k] - rest;
        const _Float16 other = (_Float16)(rest - error);
        const bool swap = error * off > 0.f && (float)other == rest - error;
        l[k] = swap ? other : l[k];
        off += swap ? -error : error;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        hi[k] = __builtin_bit_cast(uint32_t, f16x2{h[2 * k], h[2 * k + 1]});
        lo[k] = __builtin_bit_cast(uint32_t, f16x2{l[2 * k], l[2 * k + 1]});
    }
}
__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// hi*hi and the cross terms as one sum
__device__ __forceinline__ float joined(float main, float cross) { return __builtin_fmaf(cross, 1.f / (1 << kLowBits), main); }

// Adds, on the fp32 matrix instructions, the products of one kernel tap: 32 output layers (lane j of either half: a layer)
// x 32 pixels (lane j: a pixel) over Cin input layers, two at a time (half h: the second).  w_at and x_at are the lane's byte
// offsets of layer h, or kOob for layers and pixels that are not there; the steps are the bytes between input layers.
// Straight from memory, ten to twenty times the time of the split form: us of a call as it is / with one pixel of 1e12 (its
// tiles' sums beside it are small) / with infinities in every tile: fire8 at 64 images 90 / 195 / 550, 5x5 of 96 layers at 16
// 53 / 648 / 875, first layer at 8 36 / 122 / 158, classifier at 32 39 / 40 / 219, network at 64 750 / 1350 / 1590.
__device__ __forceinline__ f32x16 plain_tap(f32x16 acc, rsrc_t rw, uint32_t w_at, uint32_t w_step, rsrc_t rx, uint32_t x_at, uint32_t x_step, int Cin, int h)
{
    for (int c0 = 0; c0 < Cin; c0 += 16) {
        float w[8], x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t c = (uint32_t)(c0 + 2 * k);
            const bool there = (int)c + h < Cin;
            w[k] = buf_ld(rw, there ? w_at : kOob, c * w_step);
            x[k] = buf_ld(rx, there ? x_at : kOob, c * x_step);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) acc = Mfma<32>::run(w[k], x[k], acc);
    }
    return acc;
}

}  // namespace split
}  // namespace sq
