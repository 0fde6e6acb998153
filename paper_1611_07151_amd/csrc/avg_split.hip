// 1x1 convolution followed by a global average pooling (the classifier) on the f16 matrix instructions, both operands as
// two f16 values each (split_common.h).  The convolution writes per-image plane sums of its results per tile of 96 pixels
// instead of the results; avg_softmax() adds them up.
//
// A wavefront owns 32 output layers x 96 pixels: per 16 input layers nine MFMAs (288 cycles) against 2 KB of kernels
// through the L1 and 6 KB of pixels from LDS, 28 of 64 and 85 of 128 bytes per cycle for a CU's four SIMDs.  The
// workgroup's wavefronts share the pixels, which are staged CK input layers at a time: the next CK are on their way in
// registers while these are multiplied.  Each pixel has a scale of its own, from the largest magnitude met so far; where
// a later part of its layers needs a smaller one, its sums are brought down to that.
// 512 -> 1000 layers at 13 x 13, launch alone, fp32 instructions / this: 32 images 62 / 26 us (660 TFLOP/s issued), 64
// images 102 / 51.  Tiles of 64 pixels with four wavefronts per SIMD are no faster (27 and 47 us): what is left
// above the MFMAs' own time (11 us at 32 images) is not latency.
#include "split_common.h"

#include <algorithm>

namespace sq {
namespace split {

constexpr int kPix = 96;                   // pixels of a tile

struct AvgParams {
    const float *in;          // fp32 map [N][Cin][HW]
    const u32x4 *wk;          // kernels from split_kernels(), their layers' words, bias or nullptr, the kernels as given
    const int *sk;
    const float *b, *raw;
    float *sums;              // [tiles][slots][Cout]: plane sums of the images a tile touches
    uint32_t in_bytes;
    int Cin, HW, PT, G, Cout, slots, tiles, gy;
    FastDiv dHW, dgy;
};

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void avg_split_kernel(const AvgParams p)
{
    constexpr int CK = 16 * WAVES, NT = 64 * WAVES, STEPS = CK / 16, D = 4, PER = 3;
    static_assert(CK / 8 * kPix == PER * NT && STEPS % D == 0, "");
    constexpr int plane = CK / 8 * kPix;
    __shared__ u32x4 patch[2 * plane];                        // [hi, lo][CK / 8][96][8 layers]
    __shared__ uint32_t top[kPix];                            // largest magnitude of a pixel so far
    __shared__ int odd_tile;                                  // an infinity or NaN among them
    __shared__ int wide_pixel[kPix];                          // its layers are spread wide

    const int t = threadIdx.x, lane = t & 63, j = lane & 31, h = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int id = xcd_remap((int)blockIdx.x, p.tiles * p.gy);       // the workgroups of a tile share an L2
    const int tile = fdiv(id, p.dgy), p0 = tile * kPix;
    const int mb = min((id - tile * p.gy) * WAVES + wv, (p.Cout + 31) / 32 - 1);
    const bool mine = (id - tile * p.gy) * WAVES + wv == mb;

    const u32x4 *const at = p.wk + (size_t)mb * p.G * 128 + lane;
    u32x4 a[D][2];
#pragma unroll
    for (int r = 0; r < D; ++r) { a[r][0] = at[r * 128]; a[r][1] = at[r * 128 + 64]; }

    const rsrc_t rin = make_rsrc(p.in, p.in_bytes);
    uint32_t off[PER];
    int q[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int e = t + k * NT, cb = e / kPix;
        q[k] = e - cb * kPix;
        const int gp = p0 + q[k], n = fdiv(gp, p.dHW);
        off[k] = gp < p.PT ? (uint32_t)((n * p.Cin + cb * 8) * p.HW + gp - n * p.HW) * 4u : kOob;
    }
    float v[PER][8];
    Range range[PER];                                         // of the layers a thread has staged of its pixels
    f32x16 main[3], cross[3];
    int es[3] = {127, 127, 127};
#pragma unroll
    for (int pb = 0; pb < 3; ++pb)
#pragma unroll
        for (int k = 0; k < 16; ++k) main[pb][k] = cross[pb][k] = 0.f;
    // the layers in v: scales, sums of the layers before to the new scale, patch
    auto stage = [&]() {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            range[k].add8(v[k]);
            atomicMax(&top[q[k]], range[k].top_bits());
        }
        __syncthreads();                   // (nobody reads the patch any more either)
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            u32x4 hi, lo;
            const uint32_t m = top[q[k]];
            if (m >= kOddMagnitude) odd_tile = 1;
            else if (spread(m, range[k].low)) wide_pixel[q[k]] = 1;
            split8(v[k], pow2(scale_exponent(m)), hi, lo);
            patch[t + k * NT] = hi;
            patch[t + k * NT + plane] = lo;
        }
#pragma unroll
        for (int pb = 0; pb < 3; ++pb) {
            const int e = scale_exponent(top[pb * 32 + j]);
            if (__ballot(e != es[pb])) {
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    main[pb][k] = __builtin_amdgcn_ldexpf(main[pb][k], e - es[pb]);
                    cross[pb][k] = __builtin_amdgcn_ldexpf(cross[pb][k], e - es[pb]);
                }
                es[pb] = e;
            }
        }
        __syncthreads();
    };
#pragma unroll
    for (int k = 0; k < PER * 8; ++k) v[k >> 3][k & 7] = buf_ld(rin, off[k >> 3], (uint32_t)((k & 7) * p.HW) * 4u);
    if (t < kPix) { top[t] = 0; wide_pixel[t] = 0; }
    if (t == 0) odd_tile = 0;
    __syncthreads();
    stage();
    // Steps of 16 layers: pixels are read one step ahead, kernels D steps, and a step asks for its share of the next layers
    // (all of them at once would stand before the kernels of later steps in the queue of loads).
    u32x4 bt[2][3][2];
    auto pixels = [&](int s, u32x4 (&b)[3][2]) {
#pragma unroll
        for (int pb = 0; pb < 3; ++pb)
#pragma unroll
            for (int r = 0; r < 2; ++r) b[pb][r] = patch[(2 * s + h) * kPix + pb * 32 + j + r * plane];
    };
    for (int c0 = 0; c0 < p.Cin; c0 += CK) {
        const bool more = c0 + CK < p.Cin;
        const u32x4 *const w = at + (size_t)(c0 >> 4) * 128;
        pixels(0, bt[0]);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            if (s + 1 < STEPS) pixels(s + 1, bt[(s + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            const u32x4 (&b)[3][2] = bt[s & 1];
#pragma unroll
            for (int pb = 0; pb < 3; ++pb) cross[pb] = mma(a[s % D][1], b[pb][0], cross[pb]);
#pragma unroll
            for (int pb = 0; pb < 3; ++pb) main[pb] = mma(a[s % D][0], b[pb][0], main[pb]);
#pragma unroll
            for (int pb = 0; pb < 3; ++pb) cross[pb] = mma(a[s % D][0], b[pb][1], cross[pb]);
            __builtin_amdgcn_sched_barrier(0);
            const int ahead = s + D < STEPS || more ? s + D : s;      // (the last steps read themselves again)
            a[s % D][0] = w[ahead * 128];
            a[s % D][1] = w[ahead * 128 + 64];
            if (more) {
#pragma unroll
                for (int k = s * PER * 8 / STEPS; k < (s + 1) * PER * 8 / STEPS; ++k)
                    v[k >> 3][k & 7] = buf_ld(rin, off[k >> 3], (uint32_t)((c0 + CK + (k & 7)) * p.HW) * 4u);
            }
        }
        if (more) stage();
    }

    // ---- scales, bias, ReLU; register 4q + i = layer 8q + 4h + i
    const int ml = mb * 32 + 4 * h, mj = mb * 32 + j;
    int word[16];
    float bias[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int m = min(ml + 8 * (k >> 2) + (k & 3), p.Cout - 1);
        word[k] = p.sk[m];
        bias[k] = p.b ? p.b[m] : 0.f;
    }
    int odd = odd_tile, wide = wide_pixel[j] | wide_pixel[32 + j] | wide_pixel[64 + j];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        odd |= word[k] & kOddRow;
        wide |= word[k] & kWideRow;
    }
    // on the fp32 instructions from memory: an infinity or NaN, or sums too small for operands that are spread wide
    int again = __ballot(odd) ? 7 : 0;
    if (!again && __ballot(wide)) {
#pragma unroll
        for (int pb = 0; pb < 3; ++pb) {
            float least = kSmall;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const bool marked = wide_pixel[pb * 32 + j] || (word[k] & kWideRow);
                least = fminf(least, marked && ml + 8 * (k >> 2) + (k & 3) < p.Cout ? fabsf(main[pb][k]) : kSmall);
            }
            if (__ballot(least < kSmall)) again |= 1 << pb;
        }
    }
#pragma unroll
    for (int pb = 0; pb < 3; ++pb)
#pragma unroll
        for (int k = 0; k < 16; ++k) main[pb][k] = joined(main[pb][k], cross[pb][k]);
    if (again) {
        const rsrc_t rw = make_rsrc(p.raw, (uint32_t)(p.Cout * p.Cin) * 4u);
#pragma unroll
        for (int pb = 0; pb < 3; ++pb) {
            if (!(again >> pb & 1)) continue;
            const int gp = p0 + pb * 32 + j, n = fdiv(gp, p.dHW);
#pragma unroll
            for (int k = 0; k < 16; ++k) main[pb][k] = 0.f;
            main[pb] = plain_tap(main[pb], rw, mj < p.Cout ? (uint32_t)(mj * p.Cin + h) * 4u : kOob, 4u, rin,
                                 gp < p.PT ? (uint32_t)((n * p.Cin + h) * p.HW + gp - n * p.HW) * 4u : kOob, 4u * p.HW, p.Cin, h);
        }
    }
#pragma unroll
    for (int pb = 0; pb < 3; ++pb)
#pragma unroll
        for (int k = 0; k < 16; ++k)
            main[pb][k] = fmaxf(__builtin_amdgcn_ldexpf(main[pb][k], again >> pb & 1 ? 0 : -es[pb] - row_exponent(word[k])) + bias[k], 0.f);

    // ---- plane sums per image: over a lane's three pixels, then over 32 lanes
    const int first = fdiv(p0, p.dHW), last = fdiv(min(p0 + kPix, p.PT) - 1, p.dHW);
    int image[3];
#pragma unroll
    for (int pb = 0; pb < 3; ++pb) {
        const int gp = p0 + pb * 32 + j;
        image[pb] = gp < p.PT ? fdiv(gp, p.dHW) : -1;
    }
    for (int n = first; n <= last; ++n) {
        float *const row = p.sums + ((size_t)tile * p.slots + n - first) * p.Cout;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            float s = 0.f;
#pragma unroll
            for (int pb = 0; pb < 3; ++pb) s += image[pb] == n ? main[pb][k] : 0.f;
            s = half_wave_sum(s);
            const int m = ml + 8 * (k >> 2) + (k & 3);
            if (j == 31 && mine && m < p.Cout) row[m] = s;
        }
    }
}

}  // namespace split

using namespace split;

namespace {
bool plan_avg(const ConvArgs &a, AvgParams &p, int &waves, AvgLayout &lay)
{
    if (a.dtype != SQ_F32 || a.K != 1 || a.S != 1 || a.P != 0 || !a.relu || a.pool_H || a.cp_in || a.cp_out || a.Cin % 64) return false;
    const long long HW = (long long)a.H * a.W, PT = a.N * HW, tiles = (PT + kPix - 1) / kPix;
    if (PT * a.Cin >= kMaxBufferElems || (long long)a.Cout * a.Cin >= kMaxBufferElems) return false;
    lay.ntiles = (int)tiles; lay.WN = 1; lay.BN = kPix; lay.slots = (int)((HW + kPix - 2) / HW + 1);
    // A workgroup takes about 20 us for 512 input layers however few there are, and one with few blocks of output layers has
    // idle wavefronts.  Whole classifiers at 13 x 13, us before / now: 512 -> 1000 8 images 33.5 / 36.9 (480 tiles of 32
    // layers x 96 pixels), 12 36.1 / 37.2 (704), 16 42.3 / 37.3 (928), 24 62.1 / 37.8; 512 -> 100 64 images 33.6 / 32.6 (452),
    // 128 44.2 / 34.7 (904); 128 -> 100 128 images 21.4 / 20.5; 512 -> 10 256 images 27.9 / 37.9.
    const int blocks = (a.Cout + 31) / 32;
    if (blocks < 3 || tiles * blocks < 900) return false;
    // eight wavefronts stage 128 layers at a time: 47.0 us at 64 images of the network against 53.4 with four and 64 layers
    waves = a.Cin % 128 == 0 && blocks > 4 ? 8 : 4;
    p.gy = (blocks + waves - 1) / waves;
    if (tiles * p.gy >= (1ll << 31)) return false;
    p.in = (const float *)a.in; p.raw = (const float *)a.w; p.b = a.b;
    p.in_bytes = (uint32_t)(PT * a.Cin * 4);
    p.Cin = a.Cin; p.HW = (int)HW; p.PT = (int)PT; p.G = a.Cin / 16; p.Cout = a.Cout; p.slots = lay.slots; p.tiles = (int)tiles;
    p.dHW = make_fastdiv(p.HW); p.dgy = make_fastdiv(p.gy);
    return true;
}
}  // namespace

size_t conv_avg_split_bytes(const ConvArgs &a)
{
    AvgParams p = {};
    AvgLayout lay;
    int waves;
    return plan_avg(a, p, waves, lay) ? (size_t)lay.ntiles * lay.slots * a.Cout * sizeof(float) : 0;
}

int conv_avg_split(const ConvArgs &a, const void *kernels, float *sums, size_t sums_bytes, AvgLayout *lay)
{
    AvgParams p = {};
    int waves;
    if (!plan_avg(a, p, waves, *lay)) return SQ_ERR_UNSUPPORTED;
    const size_t bytes = (size_t)lay->ntiles * lay->slots * a.Cout * sizeof(float);
    if (sums_bytes < bytes) return SQ_ERR_WORKSPACE;
    p.wk = (const u32x4 *)kernels;
    p.sk = reinterpret_cast<const int *>((const char *)kernels + (size_t)((a.Cout + 31) / 32) * p.G * 2048);
    p.sums = sums;
    LaunchScope scope("k1s1_split_96+planesums", conv_flops(a), conv_bytes(a) - 4.0 * a.N * a.Cout * a.Ho * a.Wo + (double)bytes,
                      3.0 * 2.0 * kPix * p.tiles * 32.0 * ((a.Cout + 31) / 32) * a.Cin);
    const dim3 grid((unsigned)(p.tiles * p.gy));
    if (waves == 8) hipLaunchKernelGGL(avg_split_kernel<8>, grid, dim3(512), 0, current_stream(), p);
    else hipLaunchKernelGGL(avg_split_kernel<4>, grid, dim3(256), 0, current_stream(), p);
    return check_launch();
}

}  // namespace sq
