// fp32 convolutions (stride 1, "same" padding) on the f16 matrix instructions, each fp32 operand as two f16 values
// (split_common.h): K x K layers on their own, and the expands of a fire layer (K x K and 1x1 of one map) in one launch.
#include "split_common.h"

#include <math.h>

#include <algorithm>

namespace sq {
namespace split {

// Kernels [Cout][Cin][K][K] fp32 -> operand order [Cout/32][Cin/16][K*K][hi, lo][64 lanes][8 f16] (lane l: output layer
// 32*mb + l % 32, input layers 16*g + 8*(l/32) .. +7; layers that do not exist are zero), scaled per output layer;
// then a word per output layer (padded to 32): its scale's exponent and marks (row_word).  One workgroup per output layer; its row goes
// through LDS where it fits (row_in_lds floats), so that memory sees whole lines read and 16 bytes per store.
constexpr int kSplitLayers = 9;
struct SplitLayer {
    const float *w;
    u32x4 *wp;
    int *words;
    int Cout, Cin, KK, G;
    FastDiv dKK;
};
struct SplitList {
    SplitLayer layer[kSplitLayers];
    int first[kSplitLayers + 1];      // workgroup (row) at which a layer starts
    int row_in_lds;
};
__global__ __launch_bounds__(256) void split_kernels_kernel(const SplitList list)
{
    extern __shared__ float row_lds[];
    __shared__ uint32_t top, low;
    int l = 0;
    while ((int)blockIdx.x >= list.first[l + 1]) ++l;
    const SplitLayer &y = list.layer[l];
    const float *const w = y.w;
    u32x4 *const wp = y.wp;
    int *const words = y.words;
    const int Cout = y.Cout, Cin = y.Cin, KK = y.KK, G = y.G, row_in_lds = list.row_in_lds;
    const FastDiv dKK = y.dKK;
    const int m = (int)blockIdx.x - list.first[l], n = Cin * KK;
    const float *row = w + (size_t)m * n;
    if (threadIdx.x == 0) { top = 0; low = ~0u; }
    __syncthreads();
    Range range;
    if (m < Cout)
        for (int e0 = threadIdx.x; e0 < n; e0 += 256 * 8) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = e0 + 256 * k < n ? row[e0 + 256 * k] : 0.f;
            range.add8(v);
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (e0 + 256 * k < row_in_lds) row_lds[e0 + 256 * k] = v[k];
        }
    const uint32_t mx = wave_max(range.top_bits()), mn = wave_min(range.low);
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&top, mx);
        atomicMin(&low, mn);
    }
    __syncthreads();
    const int ex = scale_exponent(top);
    const float s = pow2(ex);
    if (threadIdx.x == 0) words[m] = row_word(ex, top, low);
    for (int e = threadIdx.x; e < G * 2 * KK; e += 256) {
        const int c8 = fdiv(e, dKK), tap = e - c8 * KK;
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int c = c8 * 8 + k, at = c * KK + tap;
            v[k] = m < Cout && c < Cin ? (at < row_in_lds ? row_lds[at] : row[at]) : 0.f;
        }
        u32x4 hi, lo;
        float off = 0.f;
        split8_kernel(v, s, hi, lo, off);
        const size_t at = ((((size_t)(m >> 5) * G + (c8 >> 1)) * KK + tap) * 2) * 64 + 32 * (c8 & 1) + (m & 31);
        wp[at] = hi;
        wp[at + 64] = lo;
    }
}

struct ExpandParams {
    const float *in;          // fp32 map [N][Cin][H][W]
    float *out;               // fp32 [N][ldc][H][W]
    const u32x4 *wk;          // K x K kernels from split_kernels_kernel, their layers' words, bias or nullptr
    const int *sk;
    const float *bk;
    const float *raw;         // the K x K kernels as given
    const float *w1, *b1;     // 1x1 kernels [Cout1][Cin] fp32 of the same input (fire layers), or nullptr
    int N, Cin, H, W, HW, PT, K, P, G, relu;
    int Cout, coff, Cout1, coff1, ldc;
    int pitch, VH;            // W + P, H + P: rows and images share their zero padding
    int TP;                   // pixels of the staged patch (padding included), the most a tile needs
    int CK;                   // input layers staged at a time (a multiple of 16)
    int pg, cwn, kg;          // a workgroup's wavefronts: pixel groups (of 32 * PB) x blocks of output layers side by side x parts of the contraction
    int tiles;
    int patch_elems;          // 16-byte elements of LDS set aside for the patch (or the sums of a split contraction)
    FastDiv dHW, dW, dPitch, dVH, dTP;
};

// The contraction of one block of 32 output layers with the staged patch: per group of 16 input layers K * K steps, one
// per tap.  Kernels come from memory (L2) D steps ahead in the ring `a`, which holds the first D steps of `at` on entry
// and the first D of `nxt`, the block that follows, on return; pixels come from LDS one step ahead.  All taps of a
// group are unrolled: their LDS offsets are a register per kernel row plus immediates, and a step costs a scalar
// instruction or two beside its loads and MFMAs (with the position of each step computed by counters and branches, 40
// scalar instructions a step, a wavefront alone on its SIMD took 620 cycles for 192 cycles of MFMAs).
template <int K, int D, int PB>
__device__ __forceinline__ void contract(f32x16 (&main)[PB], f32x16 (&cross)[PB], u32x4 (&a)[D][2], const u32x4 *at, const u32x4 *nxt, int G,
                                         int pitch, const u32x4 *patch, int plane, int TP, const int (&lane_pix)[PB], int lane)
{
    constexpr int KK = K * K;
    static_assert(KK % D == 0, "the ring position of a step is known at compile time");
    u32x4 b[2][PB][2];
    int base[PB][2], row[PB][2];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        base[pb][0] = row[pb][0] = lane_pix[pb];
        base[pb][1] = row[pb][1] = lane_pix[pb] + plane;
        b[0][pb][0] = patch[row[pb][0]];
        b[0][pb][1] = patch[row[pb][1]];
    }
    for (int g = 0; g < G; ++g) {
        const u32x4 *const pn = g + 1 < G ? at + KK * 128 : nxt;
        const int step = g + 1 < G ? 2 * TP : 0;       // (the last group reads ahead into itself)
#pragma unroll
        for (int r = 0; r < KK; ++r) {
            const int cur = r & 1;
#pragma unroll
            for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (r + 1 == KK) row[pb][q] = base[pb][q] = base[pb][q] + step;
                    else if ((r + 1) % K == 0) row[pb][q] += pitch;
                    b[cur ^ 1][pb][q] = patch[row[pb][q] + (r + 1 == KK ? 0 : (r + 1) % K)];
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) cross[pb] = mma(a[r % D][1], b[cur][pb][0], cross[pb]);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) main[pb] = mma(a[r % D][0], b[cur][pb][0], main[pb]);
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) cross[pb] = mma(a[r % D][0], b[cur][pb][1], cross[pb]);
            const u32x4 *const src = r + D < KK ? at + (r + D) * 128 : pn + (r + D - KK) * 128;
            a[r % D][0] = src[lane];
            a[r % D][1] = src[64 + lane];
            __builtin_amdgcn_sched_barrier(0);
        }
        at = pn;
        if constexpr (KK & 1)
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) { b[0][pb][0] = b[1][pb][0]; b[0][pb][1] = b[1][pb][1]; }
    }
}

// A workgroup owns pg * 32 * PB consecutive pixels of the batch and stages what their K x K windows touch, once, as hi
// and lo planes in LDS; its wavefronts share out the blocks of 32 output layers (and, where there are too few of those
// to fill the chip, parts of the contraction, added up through LDS at the end).  The patch is a stretch of the map with
// one column of zeros between rows and P rows of zeros between images, so that a tap is a constant shift for every
// pixel, at borders too.  Bound: with 96 pixels per wavefront (PB = 3) a step of nine MFMAs (288 cycles) reads 2 KB of
// kernels through the L1 and 6 KB of pixels from LDS: 28 of 64 and 85 of 128 bytes per cycle for the four SIMDs
// together, so the matrix units are the longest part; with 32 pixels (small batches, more workgroups) the L1 is.
// PARTS: the input layers do not fit LDS at once (then every wavefront has
// one block of output layers).
template <int K, int D, int PB, bool PARTS>
__global__ __launch_bounds__(512, 2) void expand_split_kernel(const ExpandParams p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    u32x4 *const patch = reinterpret_cast<u32x4 *>(smem);
    const int plane = (p.CK >> 3) * p.TP;
    int *const rows = reinterpret_cast<int *>(patch + p.patch_elems);            // [8 wavefronts][32] words of a 1x1 block's layers
    uint32_t *const red = reinterpret_cast<uint32_t *>(rows + 8 * 32);           // [8 wavefronts][2] range of the magnitudes
    int2 *const bias = reinterpret_cast<int2 *>(red + 16);                       // [units][cwn][32] (layer's word, bias)

    const int t = threadIdx.x, lane = t & 63, nthreads = (int)blockDim.x;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6), waves = nthreads >> 6;
    const int j = lane & 31, h = lane >> 5;
    const int tile = xcd_remap((int)blockIdx.x, p.tiles);
    const int npx = p.pg * 32 * PB, p0 = tile * npx;
    const int kw = wv % p.kg, grp = wv / p.kg % p.pg, cw = wv / (p.kg * p.pg);

    // ---- blocks of output layers: unit u of this wavefront is block u * stride + first_block (units uk.. are 1x1 blocks)
    const int nbk = (p.Cout + 31) >> 5, nb1 = p.w1 ? (p.Cout1 + 31) >> 5 : 0;
    const int stride = p.cwn * (int)gridDim.y, first_block = (int)blockIdx.y * p.cwn + cw;
    const int uk = (nbk + stride - 1) / stride, u1 = (nb1 + stride - 1) / stride;

    // kernels of the first unit: asked for before the patch is staged
    u32x4 a[D][2];
    auto part = [&](int c0, int &g0, int &g1) {
        const int G = min(p.CK, p.Cin + 15 - c0) >> 4;
        g0 = kw * G / p.kg;
        g1 = (kw + 1) * G / p.kg;
    };
    auto stream = [&](int u, int c0) {
        int g0, g1;
        part(c0, g0, g1);
        const int mb = min(u * stride + first_block, nbk - 1);
        return p.wk + ((size_t)mb * p.G + (c0 >> 4) + g0) * (K * K * 128);
    };
    {
        const u32x4 *const at = stream(0, 0);
#pragma unroll
        for (int r = 0; r < D; ++r) {
            a[r][0] = at[r * 128 + lane];
            a[r][1] = at[r * 128 + 64 + lane];
        }
    }

    // position of a pixel in the padded stretch
    auto stretch = [&](int gp) {
        const int n = fdiv(gp, p.dHW), pix = gp - n * p.HW, y = fdiv(pix, p.dW), x = pix - y * p.W;
        return (n * p.VH + y + p.P) * p.pitch + x + p.P;
    };
    const int first = stretch(p0) - p.P * p.pitch - p.P;      // first staged position (>= 0)

    // ---- element e of the patch: eight layers of one position
    auto fetch = [&](int e, int c0, float (&v)[8]) {
        const int cb = fdiv(e, p.dTP), q = first + e - cb * p.TP;
        const int vr = fdiv(q, p.dPitch), x = q - vr * p.pitch - p.P;
        const int n = fdiv(vr, p.dVH), y = vr - n * p.VH - p.P;
        const int c = c0 + cb * 8;
        const bool ok = x >= 0 && y >= 0 && n < p.N;
        const float *src = p.in + ((size_t)n * p.Cin + c) * p.HW + y * p.W + x;
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = ok && c + k < p.Cin ? src[(size_t)k * p.HW] : 0.f;
    };
    // ---- the patch, and the range of the magnitudes it holds
    const int items = (p.CK >> 3) * p.TP;
    constexpr int kKeep = PARTS ? 0 : 10;                      // elements a thread holds from the scan to the split
    uint32_t mx, mn;
    auto put = [&](int e, const float (&v)[8], float s) {
        u32x4 hi, lo;
        split8(v, s, hi, lo);
        patch[e] = hi;
        patch[e + plane] = lo;
    };
    auto stage = [&](int e0, int c0, float s) {
        for (int e = e0; e < items; e += nthreads) {
            float v[8];
            fetch(e, c0, v);
            put(e, v, s);
        }
    };
    {
        float kept[kKeep + 1][8];
        Range range;
#pragma unroll
        for (int k = 0; k < kKeep; ++k)
            if (t + k * nthreads < items) fetch(t + k * nthreads, 0, kept[k]);
        // words and bias of this workgroup's layers (those of the 1x1 kernels are found with the kernels)
        for (int e = t; e < (uk + u1) * p.cwn * 32; e += nthreads) {
            const int u = e / (p.cwn * 32), c = (e >> 5) - u * p.cwn;
            const bool one = u >= uk;
            const int m = ((one ? u - uk : u) * stride + (int)blockIdx.y * p.cwn + c) * 32 + (e & 31);
            const float *b = one ? p.b1 : p.bk;
            bias[e] = int2{!one && m < p.Cout ? p.sk[m] : 0, b && m < (one ? p.Cout1 : p.Cout) ? __builtin_bit_cast(int, b[m]) : 0};
        }
#pragma unroll
        for (int k = 0; k < kKeep; ++k)
            if (t + k * nthreads < items) range.add8(kept[k]);
        for (int c0 = 0; c0 < p.Cin; c0 += p.CK)
            for (int e = t + kKeep * nthreads; e < items; e += nthreads) {
                float v[8];
                fetch(e, c0, v);
                range.add8(v);
            }
        mx = wave_max(range.top_bits());
        mn = wave_min(range.low);
        if (lane == 0) { red[2 * wv] = mx; red[2 * wv + 1] = mn; }
        __syncthreads();
        for (int k = 0; k < waves; ++k) { mx = max(mx, red[2 * k]); mn = min(mn, red[2 * k + 1]); }
        mx = __builtin_amdgcn_readfirstlane(mx);
        mn = __builtin_amdgcn_readfirstlane(mn);
        if (!PARTS) {
            const float s = pow2(scale_exponent(mx));
#pragma unroll
            for (int k = 0; k < kKeep; ++k)
                if (t + k * nthreads < items) put(t + k * nthreads, kept[k], s);
            stage(t + kKeep * nthreads, 0, s);
            __syncthreads();
        }
    }
    const int es = scale_exponent(mx);
    const bool odd = mx >= kOddMagnitude, wide = spread(mx, mn);

    // ---- this wavefront's pixels
    int lane_pix[PB];
    uint32_t obase[PB];
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
        const int gp = p0 + (grp * PB + pb) * 32 + j;
        const int gq = gp < p.PT ? gp : p0;
        lane_pix[pb] = stretch(gq) - p.P * p.pitch - p.P - first + h * p.TP;
        const int n = fdiv(gq, p.dHW);
        obase[pb] = gp < p.PT ? (uint32_t)((n * p.ldc + 4 * h) * p.HW + gq - n * p.HW) * 4u : kOob;
    }
    const rsrc_t rout = make_rsrc(p.out, (uint32_t)((size_t)p.N * p.ldc * p.HW * 4));
    const float lowest = p.relu ? 0.f : -__builtin_inff();

    // ---- a block of 32 output layers on the fp32 instructions, from memory, for those pixel blocks that `which` names
    auto plain = [&](int which, const float *w, int taps, int mb, int Cout, int coff, const int2 *sb) {
        const int side = taps == 1 ? 1 : K, reach = side / 2, m = mb * 32 + j;
        const rsrc_t rw = make_rsrc(w, (uint32_t)(Cout * p.Cin * taps) * 4u), rx = make_rsrc(p.in, (uint32_t)((size_t)p.N * p.Cin * p.HW * 4));
        const uint32_t wo = (uint32_t)((m * p.Cin + h) * taps) * 4u;
#pragma unroll 1
        for (int pb = 0; pb < PB; ++pb) {
            if (!(which >> pb & 1)) continue;
            const int gp = p0 + (grp * PB + pb) * 32 + j, gq = min(gp, p.PT - 1), n = fdiv(gq, p.dHW), pix = gq - n * p.HW, y = fdiv(pix, p.dW), x = pix - y * p.W;
            f32x16 sum;
#pragma unroll
            for (int k = 0; k < 16; ++k) sum[k] = 0.f;
#pragma unroll 1
            for (int tap = 0; tap < taps; ++tap) {
                const int yy = y + tap / side - reach, xx = x + tap % side - reach;
                const bool inside = yy >= 0 && yy < p.H && xx >= 0 && xx < p.W;
                sum = plain_tap(sum, rw, m < Cout ? wo + 4u * tap : kOob, 4u * taps, rx, inside ? (uint32_t)((n * p.Cin + h) * p.HW + yy * p.W + xx) * 4u : kOob,
                                4u * p.HW, p.Cin, h);
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int ml = 8 * (k >> 2) + 4 * h + (k & 3);
                if (gp < p.PT && mb * 32 + ml < Cout)
                    p.out[((size_t)n * p.ldc + coff + mb * 32 + ml) * p.HW + pix] = fmaxf(sum[k] + __builtin_bit_cast(float, sb[ml].y), lowest);
            }
        }
    };

    // ---- remove the scales, bias, ReLU; register 4q + i = layer 8q + 4h + i: 32 neighbouring pixels per store
    auto finish = [&](f32x16 (&main)[PB], f32x16 (&cross)[PB], int mb, int Cout, int coff, const int2 *sb, const int *words, const float *w, int taps) {
        const int word = words ? words[j] : sb[j].x;
        int again = odd || __ballot(word & kOddRow) ? (1 << PB) - 1 : 0;
        if (!again && (wide || __ballot(word & kWideRow))) {
#pragma unroll
            for (int pb = 0; pb < PB; ++pb) {
                float least = kSmall;
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const int ml = 8 * (k >> 2) + 4 * h + (k & 3);
                    const bool marked = wide || ((words ? words[ml] : sb[ml].x) & kWideRow);
                    least = fminf(least, marked && mb * 32 + ml < Cout ? fabsf(main[pb][k]) : kSmall);
                }
                if (__ballot(least < kSmall)) again |= 1 << pb;
            }
        }
        uint32_t at[PB];
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) at[pb] = again >> pb & 1 ? kOob : obase[pb];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int ml = 8 * q + 4 * h + i;
                const int2 f = sb[ml];
                const int ex = -es - row_exponent(words ? words[ml] : f.x);
                const uint32_t so = (uint32_t)((coff + mb * 32 + 8 * q + i) * p.HW) * 4u;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    const float v = fmaxf(__builtin_amdgcn_ldexpf(joined(main[pb][4 * q + i], cross[pb][4 * q + i]), ex) + __builtin_bit_cast(float, f.y), lowest);
                    buf_st(rout, mb * 32 + ml < Cout ? at[pb] : kOob, so, v);
                }
            }
        if (again) plain(again, w, taps, mb, Cout, coff, sb);
    };
    auto clear = [&](f32x16 (&main)[PB], f32x16 (&cross)[PB]) {
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
#pragma unroll
            for (int k = 0; k < 16; ++k) main[pb][k] = cross[pb][k] = 0.f;
    };
    for (int u = 0; u < uk; ++u) {
        const int mb = u * stride + first_block;
        f32x16 main[PB], cross[PB];
        clear(main, cross);
        for (int c0 = 0; c0 < p.Cin; c0 += p.CK) {
            if (PARTS) {
                __syncthreads();
                stage(t, c0, pow2(es));
                __syncthreads();
            }
            int g0, g1;
            part(c0, g0, g1);
            const bool more = c0 + p.CK < p.Cin;
            const u32x4 *const nxt = stream(more || u + 1 == uk ? u : u + 1, more ? c0 + p.CK : 0);
            contract<K, D, PB>(main, cross, a, stream(u, c0), nxt, g1 - g0, p.pitch, patch + 2 * g0 * p.TP, plane, p.TP, lane_pix, lane);
        }
        // parts of the contraction: added up in the order of the parts, in the patch (nobody reads it any more: a launch that
        // splits the contraction has one unit per wavefront)
        if (p.kg > 1) {
            f32x4 *const sums = reinterpret_cast<f32x4 *>(patch);
            __syncthreads();
            if (kw > 0) {
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        f32x4 v;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = joined(main[pb][4 * q + i], cross[pb][4 * q + i]);
                        sums[((wv * PB + pb) * 4 + q) * 64 + lane] = v;
                    }
            }
            __syncthreads();
            if (kw > 0) continue;
            for (int k = 1; k < p.kg; ++k)
#pragma unroll
                for (int pb = 0; pb < PB; ++pb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 v = sums[(((wv + k) * PB + pb) * 4 + q) * 64 + lane];
#pragma unroll
                        for (int i = 0; i < 4; ++i) main[pb][4 * q + i] += v[i];
                    }
        }
        if (mb < nbk) finish(main, cross, mb, p.Cout, p.coff, bias + (u * p.cwn + cw) * 32, nullptr, p.raw, K * K);
    }
    if constexpr (!PARTS) {
        // 1x1 kernels straight from memory (at most 64 input layers): lane = output layer j, eight input layers per half; the
        // loads of the next block are in flight while this one is multiplied and stored
        f32x4 w[4][2];
        auto load_w = [&](int u) {
            const int m = min(u * stride + first_block, nb1 - 1) * 32 + j;
            const float *const wr = p.w1 + (size_t)(m < p.Cout1 ? m : 0) * p.Cin + 8 * h;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float *const at = wr + 16 * (g < p.G ? g : 0);
                w[g][0] = *reinterpret_cast<const f32x4_a4 *>(at);
                w[g][1] = *reinterpret_cast<const f32x4_a4 *>(at + 4);
            }
        };
        if (u1 > 0) load_w(0);
        for (int u = 0; u < u1; ++u) {
            const int mb = u * stride + first_block;
            Range range;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float v[8] = {w[g][0].x, w[g][0].y, w[g][0].z, w[g][0].w, w[g][1].x, w[g][1].y, w[g][1].z, w[g][1].w};
                range.add8(v);
            }
            const uint32_t top = max(range.top_bits(), (uint32_t)__shfl_xor((int)range.top_bits(), 32, 64));
            const uint32_t low = min(range.low, (uint32_t)__shfl_xor((int)range.low, 32, 64));
            const int ex = scale_exponent(top);
            const float ws = pow2(ex);
            if (h == 0) rows[wv * 32 + j] = row_word(ex, top, low);
            u32x4 ah[4], al[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float v[8] = {w[g][0].x, w[g][0].y, w[g][0].z, w[g][0].w, w[g][1].x, w[g][1].y, w[g][1].z, w[g][1].w};
                split8(v, ws, ah[g], al[g]);
            }
            if (u + 1 < u1) load_w(u + 1);
            f32x16 main[PB], cross[PB];
            clear(main, cross);
            const int centre = p.P * p.pitch + p.P;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (g >= p.G) break;
#pragma unroll
                for (int pb = 0; pb < PB; ++pb) {
                    const u32x4 bh = patch[lane_pix[pb] + centre + 2 * g * p.TP], bl = patch[lane_pix[pb] + centre + 2 * g * p.TP + plane];
                    cross[pb] = mma(al[g], bh, cross[pb]);
                    main[pb] = mma(ah[g], bh, main[pb]);
                    cross[pb] = mma(ah[g], bl, cross[pb]);
                }
            }
            if (mb < nb1) finish(main, cross, mb, p.Cout1, p.coff1, bias + ((uk + u) * p.cwn + cw) * 32, rows + wv * 32, p.w1, 1);
        }
    }
}

}  // namespace split

// ------------------------------------------------------------------------------ host side
using namespace split;

size_t split_kernel_bytes(int Cout, int Cin, int K)
{
    const size_t mb = ((size_t)Cout + 31) / 32;
    return mb * K * K * (((size_t)Cin + 15) / 16) * 2048 + mb * 32 * sizeof(float);
}

int split_kernels(const SplitJob *jobs, int njobs)
{
    SplitList list = {};
    double bytes = 0;
    int rows = 0, longest = 0;
    for (int l = 0; l < njobs; ++l) {
        const SplitJob &j = jobs[l];
        const int mb = (j.Cout + 31) / 32, G = (j.Cin + 15) / 16, KK = j.K * j.K;
        list.layer[l] = SplitLayer{(const float *)j.w, (u32x4 *)j.dst, reinterpret_cast<int *>((char *)j.dst + (size_t)mb * KK * G * 2048), j.Cout, j.Cin, KK, G,
                                   make_fastdiv(KK)};
        list.first[l] = rows;
        rows += mb * 32;
        longest = std::max(longest, j.Cin * KK);
        bytes += 8.0 * j.Cout * j.Cin * KK;
    }
    for (int l = njobs; l <= kSplitLayers; ++l) list.first[l] = rows;
    list.row_in_lds = std::min(longest, 15 * 1024);
    LaunchScope scope("split_kernels", 0.0, bytes, 0.0);
    hipLaunchKernelGGL(split_kernels_kernel, dim3(rows), dim3(256), list.row_in_lds * sizeof(float), current_stream(), list);
    return check_launch();
}

int split_kernels(const float *w, void *dst, int Cout, int Cin, int K)
{
    const SplitJob job = {w, dst, Cout, Cin, K};
    return split_kernels(&job, 1);
}

namespace {

typedef void (*ExpandFn)(const ExpandParams);
template <bool PARTS> ExpandFn expand_fn(int K, int PB)
{
    if (K == 3) return PB == 3 ? expand_split_kernel<3, 3, 3, PARTS> : expand_split_kernel<3, 9, 1, PARTS>;
    return PB == 3 ? expand_split_kernel<5, 5, 3, PARTS> : expand_split_kernel<5, 5, 1, PARTS>;
}
ExpandFn expand_fn(int K, int PB, bool parts) { return parts ? expand_fn<true>(K, PB) : expand_fn<false>(K, PB); }

// pixels of the padded stretch that the windows of npx consecutive pixels touch, at most
long long stretch_pixels(int npx, int H, int W, int P)
{
    const long long rows = npx >= 2 ? (npx - 2) / W + 2 : 1;
    const long long images = rows >= 2 ? (rows - 2) / H + 1 : 0;      // image borders among them
    return npx + (rows - 1) * P + images * (long long)P * (W + P) + 2ll * ((long long)P * (W + P) + P);
}

constexpr size_t kExpandFixed = 8 * 32 * 4 + 16 * 4;

struct ExpandPlan {
    ExpandParams p;
    int PB, waves, gy;
    bool parts;
    size_t lds;
};

// a1: the 1x1 layer of the same map, or nullptr
bool plan_expand(const ConvArgs &a, const ConvArgs *a1, const void *wk, ExpandPlan &pl, bool kg_allowed = true)
{
    if (a.dtype != SQ_F32 || (a.K != 3 && a.K != 5) || a.S != 1 || a.P != (a.K - 1) / 2 || a.pool_H || a.cp_in || a.cp_out) return false;
    if (a1 && (a.Cin % 16 || a.Cin > 64)) return false;
    const long long PT = (long long)a.N * a.H * a.W;
    if ((long long)a.N * a.Cin * a.H * a.W >= kMaxBufferElems || (long long)a.N * a.out_channels * a.H * a.W >= kMaxBufferElems ||
        (long long)(a.H + a.P) * (a.W + a.P) * (a.N + 1ll) >= (1ll << 30) || (long long)a.Cout * a.Cin * a.K * a.K >= kMaxBufferElems)
        return false;
    ExpandParams &p = pl.p;
    p.in = (const float *)a.in; p.out = a.out; p.wk = (const u32x4 *)wk; p.raw = (const float *)a.w; p.bk = a.b;
    p.N = a.N; p.Cin = a.Cin; p.H = a.H; p.W = a.W; p.HW = a.H * a.W; p.PT = (int)PT; p.K = a.K; p.P = a.P; p.G = (a.Cin + 15) / 16;
    p.relu = a.relu; p.Cout = a.Cout; p.coff = a.c_offset; p.ldc = a.out_channels;
    p.w1 = a1 ? (const float *)a1->w : nullptr; p.b1 = a1 ? a1->b : nullptr; p.Cout1 = a1 ? a1->Cout : 0; p.coff1 = a1 ? a1->c_offset : 0;
    const int nb = (a.Cout + 31) / 32;
    p.sk = reinterpret_cast<const int *>((const char *)wk + (size_t)nb * a.K * a.K * p.G * 2048);
    p.pitch = a.W + a.P; p.VH = a.H + a.P;
    p.dHW = make_fastdiv(p.HW); p.dW = make_fastdiv(a.W); p.dPitch = make_fastdiv(p.pitch); p.dVH = make_fastdiv(p.VH);

    // Tile and share of the wavefronts.  A wavefront's own tile is 32 output layers x 96 pixels where at least 1900
    // tiles of 32 x 32 are there (two per SIMD) and the patch fits LDS whole, else 32 x 32.  Measured around that line on the network's expands, us with 32 / 96 pixels: 16 -> 64 at 55x55 1512 tiles
    // 14.8 / 15.9, 3025 tiles 21.8 / 17.7; 48 -> 192 at 27x27 1093 tiles 17.4 / 20.7, 2187 tiles 27.2 / 22.0; 64 -> 256 at
    // 27x27 1458 tiles 20.8 / 22.9, 2916 tiles 31.3 / 25.2; 96 -> 256 of 5x5 at 27x27 2916
    // tiles 65.1 / 45.3; with 256 input layers at 13x13 (in two parts) 4056 tiles 70.8 / 111.9.  (64 pixels are never the best of the three by more than the noise.)  Where even 32 x 32 leaves some
    // of the 4 SIMDs of every CU without a tile, the input layers are dealt out too, to up to four wavefronts.
    pl.waves = 4;
    const long long simds = 4ll * num_cus();
    auto tiles_of = [&](long long npx) { return (PT + npx - 1) / npx; };
    pl.PB = tiles_of(32) * nb >= 1900 && stretch_pixels(96, a.H, a.W, a.P) * p.G * 64 <= kLdsBytes - 16 * 1024 ? 3 : 1;
    p.kg = 1;
    while (kg_allowed && p.kg < 4 && 2 * p.kg <= p.G && !a1 && tiles_of(32 * pl.PB) * nb * p.kg < simds) p.kg *= 2;
    // eight wavefronts around one patch where two workgroups of four would not fit a CU's LDS side by side
    const long long patch64 = stretch_pixels(32 * pl.PB, a.H, a.W, a.P) * p.G * 16 * 4;
    if (nb * p.kg >= 8 && 2 * (patch64 + 4096) > kLdsBytes) pl.waves = 8;
    int per = pl.waves / p.kg;                                          // pixel groups x layer blocks of a workgroup
    p.pg = per > 1 && (nb % per) != 0 ? 2 : 1;
    if (nb < 2) p.pg = per;
    p.cwn = per / p.pg;
    const long long groups = (nb + p.cwn - 1) / p.cwn;
    const int npx = 32 * pl.PB * p.pg;
    const long long tiles = tiles_of(npx), TP = stretch_pixels(npx, a.H, a.W, a.P);
    if (TP > (1 << 20) || tiles >= (1ll << 31)) return false;
    const long long per_layer = 2 * TP * 2;                             // bytes of LDS per input layer
    const long long room = kLdsBytes - 16 * 1024;
    pl.parts = p.G * 16 * per_layer > room;
    p.CK = p.G * 16;
    if (pl.parts) {
        if (a1) return false;
        const int parts = (int)((p.G * 16 * per_layer + room - 1) / room);
        p.CK = (p.G + parts - 1) / parts * 16;
        if (p.CK * per_layer > room) p.CK -= 16;
        if (p.CK < 16) return false;
        // (every part of a split contraction needs steps in the last, smaller chunk too)
        const int last = p.G * 16 % p.CK;
        if (p.kg > 1 && (p.CK < 16 * p.kg || (last && last < 16 * p.kg))) return plan_expand(a, a1, wk, pl, false);
    }
    pl.gy = (int)((nb + p.cwn - 1) / p.cwn);
    if (!pl.parts && p.kg == 1) {   // several blocks per wavefront share the staged patch where there are workgroups enough
        const long long gy = (2ll * num_cus() + tiles - 1) / tiles;
        pl.gy = (int)std::min<long long>(groups, std::max<long long>(1, gy));
    }
    const int stride = p.cwn * pl.gy;
    const long long units = (nb + stride - 1) / stride + (a1 ? ((a1->Cout + 31) / 32 + stride - 1) / stride : 0);
    if (pl.gy > 65535) return false;
    p.TP = (int)TP; p.dTP = make_fastdiv(p.TP); p.tiles = (int)tiles;
    const size_t patch = std::max<size_t>((size_t)p.CK * per_layer, p.kg > 1 ? (size_t)pl.waves * 4096 * pl.PB : 0);
    p.patch_elems = (int)(patch / 16);
    pl.lds = patch + kExpandFixed + units * p.cwn * 32 * 8;
    return pl.lds <= (size_t)kLdsBytes;
}

// Time of a planned launch in us, with that of its kernels' split for a layer on its own: turns of a CU with one workgroup
// and with two, each with its contraction steps, the staging of its patch (read twice where it is staged in parts) and its
// stores.  Fitted to 3000 layers and 1500 fire layers' expands (16 to 512 input layers, maps of 7 to 56 pixels, 1 to 96
// images): off by 6.5 % (root mean square).
double expand_us(const ExpandPlan &pl)
{
    const ExpandParams &p = pl.p;
    const bool pair = p.w1 != nullptr;
    const double taps = p.K * p.K + (pair ? 1 : 0), nb = (p.Cout + 31) / 32, simd_waves = pl.waves / 4.0, units = ceil(nb / (p.cwn * pl.gy));
    const bool two = 2 * pl.lds <= (size_t)kLdsBytes && pl.waves == 4;
    const double turns = ceil((double)p.tiles * pl.gy / num_cus()), full = two ? floor(turns / 2) : 0.0, single = turns - 2 * full;
    const double steps = units * p.G * taps / p.kg * pl.PB * simd_waves, staged = p.TP * p.G * 0.016 / simd_waves * (pl.parts ? 2 : 1);
    const double us = (pair ? 9.0 : 10.0 + 2.46e-2 * nb * p.G * taps / 9) + single * (0.072 * steps + 0.307 * staged) + full * (0.136 * steps + 0.349 * staged) +
                      (single + full) * 0.64 * units * pl.PB * simd_waves * (pair ? 2 : 1);
    return pair ? us : std::max(13.2, us);
}

int launch_expand(const ExpandPlan &pl, const ConvArgs &a, const ConvArgs *a1)
{
    ExpandFn fn = expand_fn(a.K, pl.PB, pl.parts);
    if (!allow_big_lds((const void *)fn)) {
        const int rc = check_launch();
        return rc ? rc : SQ_ERR_HIP;
    }
    static const char *const names[2][2][2] = {{{"k3s1_split_32", "k3s1_split_96"}, {"k5s1_split_32", "k5s1_split_96"}},
                                               {{"k3s1_split_32+k1", "k3s1_split_96+k1"}, {"", ""}}};
    const double px = 32.0 * pl.PB * pl.p.pg * pl.p.tiles * 2.0 * 3.0 * 16.0 * pl.p.G;
    const double issued = px * (32.0 * ((a.Cout + 31) / 32) * a.K * a.K + (a1 ? 32.0 * ((a1->Cout + 31) / 32) : 0.0));
    LaunchScope scope(names[a1 != nullptr][a.K == 5][pl.PB > 1], conv_flops(a) + (a1 ? conv_flops(*a1) : 0.0),
                      conv_bytes(a) + (a1 ? conv_bytes(*a1) - 4.0 * a.N * a.Cin * a.H * a.W : 0.0), issued);
    hipLaunchKernelGGL(fn, dim3((unsigned)pl.p.tiles, (unsigned)pl.gy), dim3(64 * pl.waves), pl.lds, current_stream(), pl.p);
    return check_launch();
}

thread_local int g_conv_split = -1;
}  // namespace

extern "C" void sq_tune_conv_split(int mode) { g_conv_split = mode < 0 ? -1 : mode ? 1 : 0; }

// Which layers on their own run in this form.  5x5 from 16 input layers on: all (1500 shapes, 0.96 to 14.8 times as fast as the
// fp32 tilings).  3x3 from 16 on, where the estimate is 15 % below that of the other kernels, and 5x5 below 16 (a group
// is 16, the rest padding), where it is below.  The launch that splits the kernels makes 3x3 layers lose below some 15 us;
// those with few output layers over many input layers do at any size (with every such layer here: 384 -> 64 at 56x56, 16
// images 125 us in the minimal-filtering form, 551 in this one; 64 -> 64 at 56x56 30 / 46).  Of 3060 3x3 shapes by
// this rule 0.5 % lose over 3 %, and the mean gain is 1.28 of the 1.30 that the better of the two would give each time.
int conv_split(const ConvArgs &a, int *variant)
{
    ExpandPlan pl;
    if (!g_conv_split) return SQ_ERR_UNSUPPORTED;
    if (!a.ws || ((uintptr_t)a.ws & 255) || a.ws_bytes < split_kernel_bytes(a.Cout, a.Cin, a.K)) return SQ_ERR_UNSUPPORTED;
    if (!plan_expand(a, nullptr, a.ws, pl)) return SQ_ERR_UNSUPPORTED;
    if (g_conv_split < 0 && (a.K == 3 ? a.Cin < 16 || expand_us(pl) > 0.85 * conv_mfma_us(a, variant) : a.Cin < 16 && expand_us(pl) > conv_mfma_us(a, variant)))
        return SQ_ERR_UNSUPPORTED;
    const int rc = split_kernels((const float *)a.w, a.ws, a.Cout, a.Cin, a.K);
    return rc ? rc : launch_expand(pl, a, nullptr);
}

// Whether the expands of a fire layer of this shape run on split operands at any batch; the kernels of the expand3x3 are then packed
// by split_kernels().  From 48 input layers on: whole fire layers with packed kernels, us before / now, 48 -> 192 at 27x27
// 20.7 / 17.3 at 3 images, 30.6 / 24.0 at 12, 37.0 / 37.7 at 24; 64 -> 256 at 27x27 33.0 / 20.0, 40.7 / 33.5, 61.2 / 47.8.
// With 16 or 32 input layers the minimal-filtering pair is as fast or faster at half of the batches (16 -> 64 at 55x55
// 14.4 / 16.0 at 6 images, 20.1 / 21.2 at 16; 32 -> 128 at 27x27 20.0 / 21.2 at 16): their contraction is too short for
// the patch that has to be split first.
bool expand_split_shape(int Csq, int Ce3) { return Csq % 16 == 0 && Csq >= 48 && Csq <= 64 && Ce3 % 32 == 0; }

// Whether it does in a fire layer called on its own: by estimate.  Of 1500 such shapes 5 % lost over 3 %, up to 38 % (64 -> 96
// at 40x40, 48 images 57 / 92 us: three blocks of layers for four wavefronts; 48 -> 192 at 28x28, 64 images 57 / 65), with
// the rule (7 % below the pair's estimate) 1.2 %, the worst 12 %; the mean gain is 1.18 without and 1.17 with it.
bool expand_split_pays(const ConvArgs &a3, const ConvArgs &a1)
{
    ExpandPlan pl;
    if (!g_conv_split || !plan_expand(a3, &a1, nullptr, pl)) return false;
    return g_conv_split > 0 || expand_us(pl) < 0.93 * expand_pair_us(a3, a1);
}

int expand_split(const ConvArgs &a3, const ConvArgs &a1, const void *packed_e3)
{
    ExpandPlan pl;
    void *const wk = packed_e3 ? const_cast<void *>(packed_e3) : a3.ws;
    if (!wk || ((uintptr_t)wk & 255) || (!packed_e3 && a3.ws_bytes < split_kernel_bytes(a3.Cout, a3.Cin, 3))) return SQ_ERR_UNSUPPORTED;
    if (!plan_expand(a3, &a1, wk, pl)) return SQ_ERR_UNSUPPORTED;
    const int rc = packed_e3 ? SQ_OK : split_kernels((const float *)a3.w, wk, a3.Cout, a3.Cin, 3);
    return rc ? rc : launch_expand(pl, a3, &a1);
}

bool split_register_kernels()
{
    bool ok = true;
    for (int K : {3, 5})
        for (int PB : {1, 3}) ok &= allow_big_lds((const void *)expand_fn(K, PB, false)) && allow_big_lds((const void *)expand_fn(K, PB, true));
    return ok;
}

}  // namespace sq
