// The first layer (7x7 kernels, stride 2, three input layers) on 16-bit matrix instructions, alone or together with the
// max pooling (3x3, stride 2) and the squeeze layer behind it.
//
// SPLIT: fp32 operands as two f16 values each (split_common.h); else bfloat16 operands (the reduced-precision network).
// One k-group of eight values = the seven taps of a kernel row plus a zero (SPLIT: plus what rounding the seven loses) = eight
// consecutive input pixels (SPLIT: seven, the last one twice), as in
// conv7_bf16.hip: 11 steps of v_mfma_f32_32x32x16 for the 21 kernel rows.
//
// A workgroup of eight wavefronts works on a tile of 256 pixels of the layer; a wavefront owns 32 of them, keeps their
// operands of all 11 steps in registers and goes through the three blocks of 32 output layers, whose kernels stay in LDS
// for the lifetime of the persistent workgroup: per step 2 KB (SPLIT) of LDS reads for 96 cycles of MFMAs, 85 of the 128
// bytes per cycle a CU's LDS delivers to its four SIMDs.
// POOL: the tile is 17 x 15 pixels, the windows of 8 x 7 pooled ones (a pixel at a tile's edge is computed twice: 1.16
// times the layer's arithmetic); each block of 32 layers goes through LDS, the wavefronts pool it and
// contract the pooled pixels with the squeeze kernels.  Neither the layer's map (303 MB at batch 64 in fp32) nor the
// pooled one exists in memory.
// Measured at 64 images of 224 x 224: fp32 layer with pooling and squeeze 264 us (fp32 matrix instructions, two launches) ->
// 144 us; bfloat16 92 us -> 67 us.  Eight images of 227 x 227, fp32 layer alone 77 us -> 31 us.  What SPLIT with POOL
// spends beside its MFMAs (a third of the 144 us) is the way of the sums through LDS, two barriers per block of
// layers, which the one workgroup that fits a CU's LDS does not hide.
// Ten wavefronts (two of them for the squeeze) need registers below 168 and spill: 240 us; eight at up to 256 do not.
#include "split_common.h"

#include <algorithm>

namespace sq {
namespace stem {

using namespace split;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kSteps = 11;
constexpr int kRowDw = 20;                        // dwords (pairs of columns) per patch row in LDS
constexpr int kMaxRows = 39;                      // patch rows per input layer (17 pixel rows)

template <bool SPLIT, bool POOL> struct Shape {
    static constexpr int NP = SPLIT ? 2 : 1;                          // planes
    static constexpr int TR = POOL ? 17 : 16, TC = POOL ? 15 : 16;    // pixels of the layer per tile
    static constexpr int SR = POOL ? 16 : 16, SC = POOL ? 14 : 16;    // distance between tiles
    static constexpr int PR = (TR - 1) * 2 + 7, PC = (TC - 1) * 2 + 8, PAIRS = PC / 2;
    static constexpr int WAVES = 8, THREADS = WAVES * 64;
    static constexpr int ITEMS = PR * PAIRS, PER = (ITEMS + THREADS - 1) / THREADS;   // column pairs of all three layers per thread
    static constexpr int PLANE = 3 * PR * kRowDw;                     // dwords of one plane of the patch
    static constexpr int MAP = SPLIT ? 36 : 20;                       // dwords per pixel of a block of 32 layers on its way to the pooling
    static constexpr size_t LDS = (size_t)3 * kSteps * NP * 1024 + (size_t)NP * PLANE * 4 + (POOL ? (size_t)(256 + 56) * MAP * 4 : 0) + 96 * 8 + 10 * 8 + 32 * 8 + (POOL ? 6 * NP * 1024 + (SPLIT ? 8 * 2 * 1024 : 0) : 0);
};

struct Params {
    const void *in;           // [N][3][H][W] fp32 or bfloat16
    const float *w, *b;       // SPLIT: kernels [Cout][3][7][7]; [Cout] or nullptr
    const u32x4 *wp;          // else: kernels packed as [3 blocks][11 steps][64 lanes][8] bfloat16
    const float *wsq32, *bsq; // POOL: SPLIT: squeeze kernels [Csq][96]; [Csq] or nullptr
    const u32x4 *wsq;         // else: packed as [6 steps][64 lanes][8] bfloat16
    float *out;               // fp32 NCHW [N][ldc][Ho][Wo]; POOL: the squeeze map, fp32 NCHW [N][Csq][Hp][Wp] or blocked bfloat16
    uint32_t in_bytes, out_bytes;
    int N, H, W, Ho, Wo, Hp, Wp, Cout, Csq, P, relu, ldc, coff;
    int CG, per_image, tiles;
    FastDiv dCG, dPer;
};

template <bool SPLIT> __device__ __forceinline__ f32x16 mfma16(u32x4 a, u32x4 b, f32x16 c)
{
    if constexpr (SPLIT) return mma(a, b, c);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

template <bool SPLIT, bool POOL, typename TIN>
__global__ __launch_bounds__(512, SPLIT ? 2 : 4) void stem_kernel(const Params p)
{
    using S = Shape<SPLIT, POOL>;
    constexpr int NP = S::NP;
    constexpr uint32_t ESZ = sizeof(TIN);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    u32x4 *const wl = reinterpret_cast<u32x4 *>(smem);
    uint32_t *const patch = reinterpret_cast<uint32_t *>(wl + 3 * kSteps * NP * 64);
    float *const map = reinterpret_cast<float *>(patch + NP * S::PLANE);                       // POOL: a block of 32 layers of the tile, and its pooled pixels
    float *const pooled = map + 256 * S::MAP;
    int2 *const sb = reinterpret_cast<int2 *>(map + (POOL ? (256 + 56) * S::MAP : 0));            // [96] (scale's exponent, bias)
    uint2 *const red = reinterpret_cast<uint2 *>(sb + 96);                                     // [8 wavefronts] range of the magnitudes, [8] (marks of the kernels' layers, whether squeeze kernels have marks), [9] (-, smallest magnitude of the kernels)
    int2 *const sbq = reinterpret_cast<int2 *>(red + 10);                                      // [32] of the squeeze
    u32x4 *const wq = reinterpret_cast<u32x4 *>(sbq + 32);                                     // POOL: its kernels [6][NP][64]
    f32x4 *const parts = reinterpret_cast<f32x4 *>(wq + 6 * NP * 64);                          // POOL, SPLIT: [8 wavefronts][2][64] its sums (16 layers)

    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int j = lane & 31, h = lane >> 5;
    if (t < 96) sb[t] = int2{0, p.b && t < p.Cout ? __builtin_bit_cast(int, p.b[t]) : 0};
    if (SPLIT && t == 0) { red[8] = uint2{0, 0}; red[9] = uint2{0, ~0u}; }
    if (POOL && t < 32) sbq[t] = int2{0, p.bsq && t < p.Csq ? __builtin_bit_cast(int, p.bsq[t]) : 0};
    // ---- kernels into LDS: [3 blocks][11 steps][NP][64 lanes][8]; lane l of step s = layer 32 * block + l % 32, kernel row
    // 2 s + l / 32 of the 21 (the 22nd is zero)
    if constexpr (SPLIT) {
        constexpr int kRows = 96 * 22, kPer = (kRows + S::THREADS - 1) / S::THREADS;
        float v[kPer][8];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int e = t + k * S::THREADS, m = e / 22, r = e - 22 * m;
            const bool ok = m < p.Cout && r < 21;
            const float *const at = p.w + (ok ? m * 147 + r * 7 : 0);
#pragma unroll
            for (int i = 0; i < 7; ++i) v[k][i] = ok ? at[i] : 0.f;
            v[k][7] = 0.f;
        }
        __syncthreads();
        uint32_t low = ~0u;                      // (of all layers together: marks no fewer than one by one would)
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int e = t + k * S::THREADS;
            Range range;
            range.add8(v[k]);
            low = min(low, range.low);
            if (e < kRows) atomicMax(reinterpret_cast<unsigned *>(&sb[e / 22].x), range.top_bits());
        }
        low = wave_min(low);
        if (lane == 0) atomicMin(&red[9].y, low);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int e = t + k * S::THREADS, m = e / 22, r = e - 22 * m;
            if (e >= kRows) continue;
            u32x4 hi, lo;
            float off = 0.f;
            split8_kernel(v[k], pow2(scale_exponent((uint32_t)sb[m].x)), hi, lo, off);
            // the eighth place takes what the seven kernels of the row lose together, and meets the seventh pixel once more
            const _Float16 rest = (_Float16)(off * (-1.f / (1 << kLowBits)));
            hi[3] = (hi[3] & 0xffffu) | (uint32_t)__builtin_bit_cast(uint16_t, rest) << 16;
            const int at = ((m >> 5) * kSteps + (r >> 1)) * 128 + 32 * (r & 1) + (m & 31);
            wl[at] = hi;
            wl[at + 64] = lo;
        }
        __syncthreads();
        if (t < 96) {
            const uint32_t top = (uint32_t)sb[t].x;
            const int word = row_word(scale_exponent(top), top, red[9].y);
            if (word & (kOddRow | kWideRow)) atomicOr(&red[8].x, word & (kOddRow | kWideRow));
            sb[t].x = row_exponent(word);
        }
    } else {
        for (int e = t; e < 3 * kSteps * 64; e += S::THREADS) wl[e] = p.wp[e];
    }

    const rsrc_t rin = make_rsrc(p.in, p.in_bytes), rout = make_rsrc(p.out, p.out_bytes);
    auto corner = [&](int tile, int &n, int &r0, int &c0) {
        n = fdiv(tile, p.dPer);
        const int rem = tile - n * p.per_image, rg = fdiv(rem, p.dCG);
        r0 = rg * S::SR;
        c0 = (rem - rg * p.CG) * S::SC;
    };

    // ---- staging: a thread fetches the three layers of PER pairs of columns
    float x[S::PER][3][2];
    auto fetch = [&](int tile) {
        int n, r0, c0;
        corner(tile, n, r0, c0);
        const int ih0 = 2 * r0 - p.P, iw0 = 2 * c0 - p.P;
#pragma unroll
        for (int k = 0; k < S::PER; ++k) {
            const int e = t + k * S::THREADS, r = e / S::PAIRS, q = e - r * S::PAIRS, ih = ih0 + r, iw = iw0 + 2 * q;
            const bool row = e < S::ITEMS && ih >= 0 && ih < p.H;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const uint32_t base = (uint32_t)(((n * 3 + c) * p.H + ih) * p.W + iw) * ESZ;
                x[k][c][0] = buf_ld_in<TIN>(rin, row && iw >= 0 && iw < p.W ? base : kOob, 0u);
                x[k][c][1] = buf_ld_in<TIN>(rin, row && iw + 1 >= 0 && iw + 1 < p.W ? base + ESZ : kOob, 0u);
            }
        }
    };
    // range of the magnitudes of this thread's pixels, to be joined over the workgroup
    auto scan = [&]() {
        Range range;
#pragma unroll
        for (int k = 0; k < S::PER; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) range.add2(x[k][c][0], x[k][c][1]);
        const uint32_t mx = wave_max(range.top_bits()), mn = wave_min(range.low);
        if (lane == 0) red[wv] = uint2{mx, mn};
    };
    auto range = [&](uint32_t &mx, uint32_t &mn) {
        mx = 0;
        mn = ~0u;
        for (int k = 0; k < S::WAVES; ++k) {
            const uint2 r = red[k];
            mx = max(mx, r.x);
            mn = min(mn, r.y);
        }
        mx = __builtin_amdgcn_readfirstlane(mx);
        mn = __builtin_amdgcn_readfirstlane(mn);
    };
    auto stash = [&](int es) {
        const float s = SPLIT ? pow2(es) : 1.f;
#pragma unroll
        for (int k = 0; k < S::PER; ++k) {
            const int e = t + k * S::THREADS, r = e / S::PAIRS, q = e - r * S::PAIRS;
            if (e >= S::ITEMS) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                uint32_t *const at = patch + (c * S::PR + r) * kRowDw + q;
                if constexpr (SPLIT) {
                    uint32_t hi, lw;
                    split2(x[k][c][0] * s, x[k][c][1] * s, hi, lw);
                    at[0] = hi;
                    at[S::PLANE] = lw;
                } else {
                    at[0] = pack_bf16x2(x[k][c][0], x[k][c][1]);
                }
            }
        }
    };

    // ---- a wavefront's 32 pixels of the layer, their operands from the patch
    const int px = wv * 32 + j, pxc = px < S::TR * S::TC ? px : 0;
    const int pr = pxc / S::TC, pc = pxc - pr * S::TC;
    u32x4 b[kSteps][NP];
    auto operands = [&]() {
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int e0 = 2 * s, e1 = 2 * s + 1 < 21 ? 2 * s + 1 : 20;    // the zero row may read any row of the window
            const int o0 = ((e0 / 7) * S::PR + e0 % 7) * kRowDw, o1 = ((e1 / 7) * S::PR + e1 % 7) * kRowDw;
            const uint32_t *const at = patch + 2 * pr * kRowDw + pc + (h ? o1 : o0);
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                u32x4 v = {at[q * S::PLANE], at[q * S::PLANE + 1], at[q * S::PLANE + 2], at[q * S::PLANE + 3]};
                v.w = SPLIT ? __builtin_amdgcn_perm(v.w, v.w, 0x01000100u) : v.w & 0xffffu;      // the eighth pixel is outside the window
                b[s][q] = v;
            }
        }
    };
    auto contract = [&](int cb, f32x16 &acc) {
        const u32x4 *const a = wl + cb * kSteps * NP * 64 + lane;
        u32x4 ah[2] = {a[0], a[0]}, al[2] = {a[(NP - 1) * 64], a[(NP - 1) * 64]};
        f32x16 cross;
#pragma unroll
        for (int k = 0; k < 16; ++k) cross[k] = 0.f;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            if constexpr (SPLIT) {
                ah[(s + 1) & 1] = a[(s + 1 < kSteps ? s + 1 : s) * 128];
                al[(s + 1) & 1] = a[(s + 1 < kSteps ? s + 1 : s) * 128 + 64];
                __builtin_amdgcn_sched_barrier(0);
                cross = mma(al[s & 1], b[s][0], cross);
                acc = mma(ah[s & 1], b[s][0], acc);
                cross = mma(ah[s & 1], b[s][NP - 1], cross);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                acc = mfma16<SPLIT>(a[s * 64], b[s][0], acc);
            }
        }
        if constexpr (SPLIT) {
#pragma unroll
            for (int k = 0; k < 16; ++k) acc[k] = joined(acc[k], cross[k]);
        }
    };
    // The contraction of a marked tile (no photograph is one), without its scale: where an infinity or NaN may be in it, and
    // where a sum is too small for operands that are spread wide, on the fp32 instructions from memory (two of the 147
    // products of a layer at a time).
    auto contract_marked = [&](int cb, int tile, int es, bool odd, f32x16 &acc) {
        int n, r0, c0;
        corner(tile, n, r0, c0);
        bool again = odd;
        if (!odd) {
            contract(cb, acc);
            const bool there = r0 + pr < p.Ho && c0 + pc < p.Wo;
            float least = kSmall;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int m = cb * 32 + 8 * (k >> 2) + 4 * h + (k & 3);
                least = fminf(least, there && m < p.Cout ? fabsf(acc[k]) : kSmall);
                acc[k] = __builtin_amdgcn_ldexpf(acc[k], -es - sb[m].x);
            }
            again = __ballot(least < kSmall) != 0;
        }
        if (!again) return;
        const int ih0 = 2 * (r0 + pr) - p.P, iw0 = 2 * (c0 + pc) - p.P, m = cb * 32 + j;
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[k] = 0.f;
#pragma unroll 2
        for (int s = 0; s < 74; ++s) {
            const int tap = 2 * s + h, c = tap / 49, i = tap / 7 - 7 * c, jx = tap - 7 * (tap / 7), ih = ih0 + i, iw = iw0 + jx;
            const bool ok = tap < 147 && ih >= 0 && ih < p.H && iw >= 0 && iw < p.W;
            const float v = buf_ld_in<TIN>(rin, ok ? (uint32_t)(((n * 3 + c) * p.H + ih) * p.W + iw) * ESZ : kOob, 0u);
            acc = Mfma<32>::run(tap < 147 && m < p.Cout ? p.w[m * 147 + tap] : 0.f, v, acc);
        }
    };

    // ---- POOL: the squeeze of a tile's 56 pooled pixels, two blocks of 32.  bfloat16: wavefronts 0 and 1 have a block each
    // (one order of additions, that of the layer alone).  SPLIT: a wavefront has one of the two steps of 16 layers of every
    // other block of 32 layers, and the sums of the four that share a block of pixels are added up at the end.
    const int qblk = SPLIT ? (wv >> 1) & 1 : wv & 1, qg = SPLIT ? wv & 1 : 0;
    const bool squeezer = POOL && (SPLIT || wv < 2);
    if (POOL && SPLIT) {
        if (wv < 6) {                                       // step wv of the six
            const bool ok = j < p.Csq;
            const float *const row = p.wsq32 + (ok ? j : 0) * 96 + 8 * h;
            auto eight = [&](int g, float (&v)[8]) {
                const f32x4 lo = *reinterpret_cast<const f32x4_a4 *>(row + 16 * g), hi = *reinterpret_cast<const f32x4_a4 *>(row + 16 * g + 4);
#pragma unroll
                for (int k = 0; k < 4; ++k) { v[k] = ok ? lo[k] : 0.f; v[4 + k] = ok ? hi[k] : 0.f; }
            };
            Range range;
            float v[8];
            for (int g = 0; g < 6; ++g) {
                eight(g, v);
                range.add8(v);
            }
            const uint32_t top = max(range.top_bits(), (uint32_t)__shfl_xor((int)range.top_bits(), 32, 64));
            const uint32_t low = min(range.low, (uint32_t)__shfl_xor((int)range.low, 32, 64));
            if (top >= kOddMagnitude || spread(top, low)) red[8].y = 1;
            const int e = scale_exponent(top);
            u32x4 hi, lo;
            float off = 0.f;
            for (int g = 0; g <= wv; ++g) {                 // (the errors of the steps before it with it)
                eight(g, v);
                split8_kernel(v, pow2(e), hi, lo, off);
            }
            wq[(wv * 2) * 64 + lane] = hi;
            wq[(wv * 2 + 1) * 64 + lane] = lo;
            if (h == 0 && wv == 0) sbq[j].x = e;
        }
    } else if (POOL) {
        if (t < 6 * 64) wq[t] = p.wsq[t];
    }
    const int pp = 32 * qblk + j, ppc = POOL ? min(pp, 55) : 0;
    f32x16 sum, sum_cross;           // of the squeeze; SPLIT: its cross terms
    bool plain = false;              // SPLIT: whether `parts` holds, without the scale, what steps added that no scale holds
    int sq_e = 127;                  // SPLIT: exponent of this pixel's scale, and the magnitude up to which it serves
    uint32_t sq_limit = 0;
    // 56 pooled pixels x 8 groups of four layers of a block, one per thread
    auto pool_block = [&]() {
        const int q = t >> 3, c4 = t & 7;
        if (q >= 56) return;
        const int qr = q / 7, qc = q - qr * 7;
        const float *const m0 = map + ((2 * qr) * S::TC + 2 * qc) * S::MAP + (SPLIT ? 4 : 2) * c4;
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = -__builtin_inff();
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const float *const at = m0 + (dy * S::TC + dx) * S::MAP;
                if constexpr (SPLIT) {
                    const f32x4 w = *reinterpret_cast<const f32x4 *>(at);
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], w[k]);
                } else {
                    const uint2 w = *reinterpret_cast<const uint2 *>(at);
                    v[0] = fmaxf(v[0], __builtin_bit_cast(float, w.x << 16)); v[1] = fmaxf(v[1], __builtin_bit_cast(float, w.x & 0xffff0000u));
                    v[2] = fmaxf(v[2], __builtin_bit_cast(float, w.y << 16)); v[3] = fmaxf(v[3], __builtin_bit_cast(float, w.y & 0xffff0000u));
                }
            }
        if constexpr (SPLIT)
            *reinterpret_cast<f32x4 *>(pooled + q * S::MAP + 4 * c4) = f32x4{v[0], v[1], v[2], v[3]};
        else      // (the maxima are bfloat16 values already: keeping the upper halves is exact)
            *reinterpret_cast<uint2 *>(pooled + q * S::MAP + 2 * c4) =
                uint2{(__builtin_bit_cast(uint32_t, v[0]) >> 16) | (__builtin_bit_cast(uint32_t, v[1]) & 0xffff0000u),
                      (__builtin_bit_cast(uint32_t, v[2]) >> 16) | (__builtin_bit_cast(uint32_t, v[3]) & 0xffff0000u)};
    };
    auto squeeze_block = [&](int cb, int es, bool scaled) {
        if (SPLIT && (cb == 1) != (wv >= 4)) return;
#pragma unroll
        for (int k0 = 0; k0 < (SPLIT ? 1 : 2); ++k0) {
            const int g = SPLIT ? qg : k0;
            if constexpr (SPLIT) {
                const f32x4 *const at = reinterpret_cast<const f32x4 *>(pooled + ppc * S::MAP + 16 * g + 8 * h);
                const f32x4 lo = at[0], hi = at[1];
                const u32x4 ah = wq[(2 * cb + g) * 128 + lane], al = wq[(2 * cb + g) * 128 + 64 + lane];
                float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int2 f = sb[cb * 32 + 16 * g + 8 * h + k];
                    v[k] = fmaxf(__builtin_amdgcn_ldexpf(v[k], scaled ? -es - f.x : 0) + __builtin_bit_cast(float, f.y), 0.f);
                }
                Range range;
                range.add8(v);
                uint32_t mag = range.top_bits();
                const auto tops = __builtin_amdgcn_permlane32_swap(mag, mag, false, false), lows = __builtin_amdgcn_permlane32_swap(range.low, range.low, false, false);
                mag = max((uint32_t)tops[0], (uint32_t)tops[1]);
                const uint32_t low = min((uint32_t)lows[0], (uint32_t)lows[1]);
                // The scale follows the largest magnitude met.  A step that would bring the sums before it down by 2^64 or
                // more, that holds a value below 2^-27 of that magnitude, an infinity or NaN, and every step where the
                // kernels hold such values, is added up in fp32.
                const bool up = mag > sq_limit;
                const int en = up ? scale_exponent(mag) : sq_e;
                const uint32_t made_for = up ? mag : max(sq_limit, 1u << 23) - (1u << 23);
                if (__ballot(mag >= kOddMagnitude || spread(made_for, low) || (sq_limit && sq_e - en >= 64)) || red[8].y) {
                    f32x16 add;
#pragma unroll
                    for (int k = 0; k < 16; ++k) add[k] = 0.f;
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        if (plain) {
                            const f32x4 old = parts[(wv * 2 + k) * 64 + lane];
                            add[4 * k] = old.x; add[4 * k + 1] = old.y; add[4 * k + 2] = old.z; add[4 * k + 3] = old.w;
                        }
                    const float *const w = p.wsq32 + (j < p.Csq ? j : 0) * 96 + cb * 32 + 16 * g + h, *const from = pooled + ppc * S::MAP + 16 * g + h;
#pragma unroll 2
                    for (int k = 0; k < 8; ++k) {
                        const int2 f = sb[cb * 32 + 16 * g + 2 * k + h];
                        const float u = fmaxf(__builtin_amdgcn_ldexpf(from[2 * k], scaled ? -es - f.x : 0) + __builtin_bit_cast(float, f.y), 0.f);
                        add = Mfma<32>::run(w[2 * k], u, add);
                    }
                    parts[(wv * 2) * 64 + lane] = f32x4{add[0], add[1], add[2], add[3]};
                    parts[(wv * 2 + 1) * 64 + lane] = f32x4{add[4], add[5], add[6], add[7]};
                    plain = true;
                    return;
                }
                if (__ballot(up)) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) {             // (at most 16 layers: the other registers hold none)
                        sum[k] = __builtin_amdgcn_ldexpf(sum[k], en - sq_e);
                        sum_cross[k] = __builtin_amdgcn_ldexpf(sum_cross[k], en - sq_e);
                    }
                    sq_e = en;
                    if (up) sq_limit = mag + (1u << 23);      // twice the magnitude the scale was made for: below 2^15
                }
                u32x4 bh, bl;
                split8(v, pow2(sq_e), bh, bl);
                sum_cross = mma(al, bh, sum_cross);
                sum = mma(ah, bh, sum);
                sum_cross = mma(ah, bl, sum_cross);
            } else {
                const u32x4 o = *reinterpret_cast<const u32x4 *>(pooled + ppc * S::MAP + 8 * g + 4 * h);
                sum = mfma16<SPLIT>(wq[(2 * cb + k0) * 64 + lane], o, sum);
            }
        }
    };

    const XcdShare share = xcd_share((int)blockIdx.x, (int)gridDim.x, p.tiles);
    int tile = share.first, es = 0;
    bool odd = false, marked = false;
    // scale of the patch in the registers (after scan() and a barrier), and the patch
    auto settle = [&]() {
        if constexpr (SPLIT) {
            uint32_t mx, mn;
            range(mx, mn);
            odd = mx >= kOddMagnitude || (__builtin_amdgcn_readfirstlane(red[8].x) & kOddRow);
            marked = odd || spread(mx, mn) || __builtin_amdgcn_readfirstlane(red[8].x);
            es = scale_exponent(mx);
        }
        stash(es);
    };
    // POOL, SPLIT: the squeeze map of the tile whose sums lie in LDS; wavefronts 2 q + block take registers 4q .. 4q + 3
    int last_tile = -1;
    auto emit = [&]() {
        if (last_tile < 0) return;
        const int q = wv >> 1, blk = wv & 1, px = 32 * blk + j, pxc = min(px, 55);
        if (8 * q >= p.Csq) return;
        int n, r0, c0;
        corner(last_tile, n, r0, c0);
        const int oh = r0 / 2 + pxc / 7, ow = c0 / 2 + pxc % 7;
        const uint32_t o = px < 56 && oh < p.Hp && ow < p.Wp ? (uint32_t)(((n * p.Csq + 4 * h) * p.Hp + oh) * p.Wp + ow) * 4u : kOob;
        f32x4 v = parts[((2 * blk) * 2 + q) * 64 + lane];
#pragma unroll
        for (int k = 1; k < 4; ++k) {
            const f32x4 u = parts[(((k & 1) + 2 * blk + 4 * (k >> 1)) * 2 + q) * 64 + lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] += u[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            buf_st(rout, o, (uint32_t)((8 * q + i) * p.Hp * p.Wp) * 4u, fmaxf(v[i] + __builtin_bit_cast(float, sbq[8 * q + 4 * h + i].y), 0.f));
    };
    if (tile < share.end) {
        fetch(tile);
        if (SPLIT) scan();
        __syncthreads();
        settle();
    }
    for (; tile < share.end; tile += share.step) {
        const bool more = tile + share.step < share.end;
        __syncthreads();               // the patch is complete
        const int es_now = es;
        const bool odd_now = odd, marked_now = SPLIT && marked;
        operands();
        if (more) fetch(tile + share.step);
        if constexpr (POOL) {
            if (SPLIT) emit();            // of the tile before
            if (squeezer) {
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    sum[k] = SPLIT ? 0.f : __builtin_bit_cast(float, sbq[8 * (k >> 2) + 4 * h + (k & 3)].y);
                    sum_cross[k] = 0.f;
                }
                plain = false;
                sq_e = 127;
                sq_limit = 0;
            }
        }
#pragma unroll 1
        for (int cb = 0; cb < 3; ++cb) {
            f32x16 acc;
#pragma unroll
            for (int k = 0; k < 16; ++k)      // (bfloat16: bias first, as in the other kernels on such maps)
                acc[k] = SPLIT ? 0.f : __builtin_bit_cast(float, sb[cb * 32 + 8 * (k >> 2) + 4 * h + (k & 3)].y);
            if (marked_now) contract_marked(cb, tile, es_now, odd_now, acc);
            else contract(cb, acc);
            if constexpr (POOL) {
                {
                    // registers 4q .. 4q + 3 = layers 8q + 4h .. + 3 of the block
                    float *const at = map + px * S::MAP;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float v[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = SPLIT ? acc[4 * q + i] : fmaxf(acc[4 * q + i], 0.f);
                        if constexpr (SPLIT) *reinterpret_cast<f32x4 *>(at + 8 * q + 4 * h) = f32x4{v[0], v[1], v[2], v[3]};
                        else *reinterpret_cast<uint2 *>(at + 4 * q + 2 * h) = uint2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                    }
                }
                // the next tile's patch: its magnitudes are joined at the first barrier, it is written after it (every
                // wavefront has its operands by then)
                if (SPLIT && more && cb == 0) scan();
                __syncthreads();
                pool_block();
                if (more && cb == 0) settle();
                __syncthreads();
                if (squeezer) squeeze_block(cb, es_now, !marked_now);
            } else {
                int n, r0, c0;
                corner(tile, n, r0, c0);
                const int oh = r0 + pr, ow = c0 + pc;
                const uint32_t o = oh < p.Ho && ow < p.Wo ? (uint32_t)(((n * p.ldc + p.coff + 4 * h) * p.Ho + oh) * p.Wo + ow) * 4u : kOob;
                const uint32_t plane4 = (uint32_t)(p.Ho * p.Wo) * 4u;
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int m = cb * 32 + 8 * q + 4 * h + i;
                        const int2 f = sb[m];
                        const float v = SPLIT ? __builtin_amdgcn_ldexpf(acc[4 * q + i], marked_now ? 0 : -es_now - f.x) + __builtin_bit_cast(float, f.y) : acc[4 * q + i];
                        buf_st(rout, m < p.Cout ? o : kOob, (uint32_t)(cb * 32 + 8 * q + i) * plane4, p.relu ? fmaxf(v, 0.f) : v);      // (without ReLU a NaN stays one)
                    }
                if (more && cb == 2) {
                    if (SPLIT) scan();
                    __syncthreads();      // every wavefront has its operands, the magnitudes are there
                    settle();
                }
            }
        }
        if constexpr (POOL) {
            if constexpr (SPLIT) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (8 * q < p.Csq) {
                        f32x4 v;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_ldexpf(joined(sum[4 * q + i], sum_cross[4 * q + i]), -sq_e - sbq[8 * q + 4 * h + i].x);
                        if (plain) {
                            const f32x4 add = parts[(wv * 2 + q) * 64 + lane];
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[i] += add[i];
                        }
                        parts[(wv * 2 + q) * 64 + lane] = v;
                    }
                last_tile = tile;
            } else if (squeezer) {
                int n, r0, c0;
                corner(tile, n, r0, c0);
                const int oh = r0 / 2 + ppc / 7, ow = c0 / 2 + ppc % 7;
                const uint32_t o = pp < 56 && oh < p.Hp && ow < p.Wp ? (uint32_t)((n * (p.Csq / 8) * p.Hp + oh) * p.Wp + ow) * 16u + 8u * (uint32_t)h : kOob;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (8 * q < p.Csq) {
                        float v[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = fmaxf(sum[4 * q + i], 0.f);
                        buf_st2(rout, o, (uint32_t)(q * p.Hp * p.Wp) * 16u, __builtin_bit_cast(float, pack_bf16x2(v[0], v[1])),
                                __builtin_bit_cast(float, pack_bf16x2(v[2], v[3])));
                    }
            }
        }
    }
    if constexpr (POOL && SPLIT) {
        __syncthreads();
        emit();
    }
}

typedef void (*StemFn)(const Params);

}  // namespace stem

// ------------------------------------------------------------------------------ host side
using namespace stem;

namespace {
template <bool SPLIT, bool POOL, typename TIN> int launch_stem(const Params &p, const char *name, double flops, double bytes, double issued)
{
    using S = Shape<SPLIT, POOL>;
    static_assert(S::LDS <= (size_t)kLdsBytes, "");
    const StemFn fn = stem_kernel<SPLIT, POOL, TIN>;
    if (!allow_big_lds((const void *)fn)) {
        const int rc = check_launch();
        return rc ? rc : SQ_ERR_HIP;
    }
    const long long per_cu = S::LDS * 2 <= (size_t)kLdsBytes ? 2 : 1;
    const unsigned blocks = (unsigned)std::min<long long>(p.tiles, per_cu * num_cus());
    LaunchScope scope(name, flops, bytes, issued * p.tiles * 256.0 * 96.0 * 16.0 * kSteps * 2.0);
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(S::THREADS), S::LDS, current_stream(), p);
    return check_launch();
}

template <bool POOL> bool place(Params &p, int N, int H, int W, int P, int esz)
{
    using S = Shape<true, POOL>;
    if ((long long)N * 3 * H * W * esz >= (1ll << 31)) return false;
    p.N = N; p.H = H; p.W = W; p.P = P;
    p.Ho = (H + 2 * P - 7) / 2 + 1; p.Wo = (W + 2 * P - 7) / 2 + 1;
    p.Hp = p.Ho >= 3 ? (p.Ho - 3) / 2 + 1 : 0; p.Wp = p.Wo >= 3 ? (p.Wo - 3) / 2 + 1 : 0;
    p.in_bytes = (uint32_t)((long long)N * 3 * H * W * esz);
    const int RG = POOL ? (p.Hp + 7) / 8 : (p.Ho + S::SR - 1) / S::SR;
    p.CG = POOL ? (p.Wp + 6) / 7 : (p.Wo + S::SC - 1) / S::SC;
    p.per_image = RG * p.CG;
    const long long tiles = (long long)N * p.per_image;
    if (tiles <= 0 || tiles >= (1ll << 30)) return false;
    p.tiles = (int)tiles;
    p.dCG = make_fastdiv(p.CG); p.dPer = make_fastdiv(p.per_image);
    return true;
}
}  // namespace

int conv7_split(const ConvArgs &a)
{
    Params p = {};
    if (a.dtype != SQ_F32 || a.K != 7 || a.S != 2 || a.Cin != 3 || a.Cout > 96 || a.pool_H || a.cp_in || a.cp_out) return SQ_ERR_UNSUPPORTED;
    if ((long long)a.N * a.out_channels * a.Ho * a.Wo >= kMaxBufferElems || !place<false>(p, a.N, a.H, a.W, a.P, 4)) return SQ_ERR_UNSUPPORTED;
    p.in = a.in; p.w = (const float *)a.w; p.b = a.b; p.out = a.out;
    p.out_bytes = (uint32_t)((long long)a.N * a.out_channels * a.Ho * a.Wo * 4);
    p.Cout = a.Cout; p.relu = a.relu; p.ldc = a.out_channels; p.coff = a.c_offset;
    return launch_stem<true, false, float>(p, "k7s2c3_split", conv_flops(a), conv_bytes(a), 3.0);
}

int stem_split(const float *in, const float *w, const float *b, const float *wsq, const float *bsq, float *out, int N, int H, int W, int P, int Csq)
{
    Params p = {};
    if (Csq > 16 || Csq % 8 || !place<true>(p, N, H, W, P, 4) || p.Hp <= 0 || p.Wp <= 0) return SQ_ERR_UNSUPPORTED;
    p.in = in; p.w = w; p.b = b; p.wsq32 = wsq; p.bsq = bsq; p.out = out;
    p.out_bytes = (uint32_t)((long long)N * Csq * p.Hp * p.Wp * 4);
    p.Cout = 96; p.Csq = Csq; p.relu = 1;
    const double px = (double)N * p.Ho * p.Wo, pq = (double)N * p.Hp * p.Wp;
    return launch_stem<true, true, float>(p, "k7s2c3_split+pool3s2+k1", 2.0 * 96 * (147.0 * px + Csq * pq), 4.0 * (3.0 * N * H * W + Csq * pq), 3.0);
}

int stem_bf16(const void *in, int dtype, const void *w7, const float *b, const void *wsq, const float *bsq, void *out, int N, int H, int W, int P, int Csq)
{
    Params p = {};
    const int esz = dtype == SQ_BF16 ? 2 : 4;
    if (Csq > 32 || Csq % 8 || !place<true>(p, N, H, W, P, esz) || p.Hp <= 0 || p.Wp <= 0) return SQ_ERR_UNSUPPORTED;
    p.in = in; p.wp = (const u32x4 *)w7; p.b = b; p.wsq = (const u32x4 *)wsq; p.bsq = bsq; p.out = (float *)out;
    p.out_bytes = (uint32_t)((long long)N * Csq * p.Hp * p.Wp * 2);
    p.Cout = 96; p.Csq = Csq; p.relu = 1;
    const double px = (double)N * p.Ho * p.Wo, pq = (double)N * p.Hp * p.Wp;
    const double flops = 2.0 * 96 * (147.0 * px + Csq * pq), bytes = (double)esz * 3.0 * N * H * W + 2.0 * Csq * pq;
    if (dtype == SQ_BF16) return launch_stem<false, true, uint16_t>(p, "k7s2c3b+pool3s2+k1b", flops, bytes, 1.0);
    return launch_stem<false, true, float>(p, "k7s2c3b+pool3s2+k1b", flops, bytes, 1.0);
}

bool stem_register_kernels()
{
    return allow_big_lds((const void *)stem_kernel<true, false, float>) & allow_big_lds((const void *)stem_kernel<true, true, float>) &
           allow_big_lds((const void *)stem_kernel<false, true, float>) & allow_big_lds((const void *)stem_kernel<false, true, uint16_t>);
}

}  // namespace sq
