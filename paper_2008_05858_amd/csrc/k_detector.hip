// Detector stage on the final frame (Sec. 2.2: photon noise plus the
// detector's own effects -- dark current, read-out noise, pixel response
// non-uniformity, cross-talk -- added on the synthetic echellogram).
//
// One kernel, one 64 x 48 pixel tile per workgroup (four fit a CU; 64 x 64 was
// 9% slower for want of waves, 64 x 32 7% for its border):
//  1. electrons of the tile and its one-pixel border into LDS: the mean
//     mu = G F + dark t (G the response map, 1 if absent), then the Poisson
//     draw of the pixel's own counter stream (or mu itself without shot
//     noise); border pixels are recomputed by each neighbouring tile (the
//     draw is a pure function of the pixel, so every copy is the same);
//  2. per output pixel: the 3 x 3 inter-pixel cross-talk gathered in a
//     fixed order (charge moving from a pixel to its neighbour at offset
//     (dx, dy) with weight K[dy+1][dx+1], charge leaving the chip lost),
//     read noise from a Box-Muller pair of the pixel's stream at draw block
//     2^31, then the ADC: floor(R / gain + bias + 1/2) clipped to
//     [0, 2^bits - 1], stored as uint16.
// HBM traffic is the frame and gain map read once plus the ADU written once
// (10 bytes per pixel with an FP32 frame); the sampler's FP64 and integer
// arithmetic sets the pace.  On a 9216^2 FP32 frame with every mean above 10:
// 3.71 -> 1.88 ms, from the listed trials of poisson_span() and the read noise
// taken in FP32 where that decides the ADU (its FP64 logarithm, root and
// cosine took as long as the sampler), the same ADU bit for bit.
#include "philox.h"

namespace e2e {

namespace {

constexpr int DT = 64;          // tile width
constexpr int DY = 48;          // tile height
constexpr int kGridY = 32768;   // tile rows per layer of the grid
constexpr int DH = DT + 2;      // width with the border
constexpr int DN = DH * (DY + 2);  // electrons held in LDS per tile

// Standard normal from a uniform pair, in FP32: sqrt(-2 ln u1) cos(2 pi u2) by
// the hardware logarithm and cosine (of revolutions).  *err bounds its error:
// u1 rounded to FP32 and the logarithm move ln u1 by at most 1.5e-7 plus
// 4e-7 |ln u1| (that, over the root, is the first term; the root of the change
// itself where it is larger than ln u1); rounding of u2 and the cosine move the
// product by at most 2e-6 times the root.
__device__ __forceinline__ float normal_f32(double u1, double u2, float *err)
{
    const float L = fmaxf(-1.3862943611f * __builtin_amdgcn_logf((float)u1), 0.0f);  // -2 ln u1
    const float root = __builtin_sqrtf(L);
    *err = fmaf(4e-6f, root, fminf(1e-6f * __builtin_amdgcn_rcpf(fmaxf(root, 1e-4f)), 1e-3f));
    return root * __builtin_amdgcn_cosf((float)u2);
}

struct DetArgs {
    double k[9];
    double dark, ron, gain, inv_gain, bias, top;
    double tiny;   // 1e-14 of the bias and of a step
    uint64_t seed;
    uint32_t fidx;
    int nx, ny;
};

template <typename T, bool SHOT>
__global__ __launch_bounds__(256) void k_detector(const T *__restrict__ frame,
                                                  const float *__restrict__ prnu, DetArgs a,
                                                  uint16_t *__restrict__ adu)
{
    __shared__ double el[DN];
    __shared__ PoissonLists<SHOT ? DN : 8> L;
    const int x0 = blockIdx.x * DT - 1;
    const int64_t ty = (int64_t)blockIdx.z * kGridY + blockIdx.y;
    if (ty * DY >= a.ny) return;
    const int y0 = (int)ty * DY - 1;
    const int bh = min(DY + 2, a.ny - y0 + 1);  // rows of the tile and border (the last may be off chip)
    auto on_chip = [&](int c) {
        const int gy = y0 + c / DH, gx = x0 + c % DH;
        return gx >= 0 && gx < a.nx && gy >= 0 && gy < a.ny;
    };
    auto pixel = [&](int c) { return (int64_t)(y0 + c / DH) * a.nx + (x0 + c % DH); };
    auto mean = [&](int c) {
        if (!on_chip(c)) return 0.0;
        const int64_t p = pixel(c);
        const double g = prnu ? (double)prnu[p] : 1.0;
        return fma(g, (double)frame[p], a.dark);
    };
    if constexpr (SHOT)
        poisson_span<DN>(
            bh * DH, a.seed, a.fidx, mean, [&](int c) { return (uint64_t)pixel(c); },
            [&](int c, double v) { el[c] = v; }, L);
    else
        for (int c = threadIdx.x; c < bh * DH; c += 256) el[c] = mean(c);
    __syncthreads();
    const int lx = threadIdx.x & 63, gx = x0 + 1 + lx;
    if (gx >= a.nx) return;
    for (int ly = threadIdx.x >> 6; ly < DY; ly += 4) {
        const int gy = y0 + 1 + ly;
        if (gy >= a.ny) break;
        double e = 0.0;
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
            for (int dx = -1; dx <= 1; ++dx)  // the pixel the charge comes from
                e = fma(a.k[(dy + 1) * 3 + (dx + 1)], el[(ly + 1 - dy) * DH + (lx + 1 - dx)], e);
        const int64_t p = (int64_t)gy * a.nx + gx;
        double v;
        auto adc = [&](double r) { return floor(r / a.gain + a.bias + 0.5); };
        if (a.ron > 0.0) {
            double u1, u2;
            uniform_pair(a.seed, a.fidx, (uint64_t)p, 0x80000000u, &u1, &u2);
            // the read noise in FP32 first: its ADU is the exact one unless the
            // value lies within the error bound of a step of the ADC, then
            // (one pixel in about 1e5) it is taken in FP64.  (The roundings of either
            // form go with the terms, not with their sum: a bias may cancel them.)
            float err;
            const float z = normal_f32(u1, u2, &err);
            const double eg = e * a.inv_gain;
            const double t = fma(a.ron * a.inv_gain, (double)z, eg) + a.bias + 0.5;
            v = floor(t);
            const double fr = t - v, lim = fma(a.ron * a.inv_gain, (double)err, fma(fabs(eg), 1e-14, a.tiny));
            if (!(fr > lim && fr < 1.0 - lim))
                v = adc(fma(a.ron, sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2), e));
        } else {
            v = adc(e);
        }
        v = fmin(fmax(v, 0.0), a.top);
        adu[p] = (uint16_t)v;
    }
}

template <typename T>
void launch_t(const T *frame, const float *prnu, const DetArgs &a, int shot, uint16_t *adu,
              hipStream_t s)
{
    const int rows = (a.ny + DY - 1) / DY;  // of tiles; a grid holds 65535 a dimension
    const dim3 grid((a.nx + DT - 1) / DT, rows < kGridY ? rows : kGridY, (rows + kGridY - 1) / kGridY);
    if (shot)
        hipLaunchKernelGGL((k_detector<T, true>), grid, dim3(256), 0, s, frame, prnu, a, adu);
    else
        hipLaunchKernelGGL((k_detector<T, false>), grid, dim3(256), 0, s, frame, prnu, a, adu);
}

}  // namespace

hipError_t launch_detector(const void *frame, int f64, const float *prnu, int nx, int ny,
                           double dark, int shot, const double *xtalk, double ron, double gain,
                           double bias, int bits, uint64_t seed, uint32_t fidx, uint16_t *adu,
                           hipStream_t s)
{
    if (nx <= 0 || ny <= 0) return hipSuccess;
    DetArgs a;
    for (int q = 0; q < 9; ++q) a.k[q] = xtalk[q];
    a.dark = dark;
    a.ron = ron;
    a.gain = gain;
    a.inv_gain = 1.0 / gain;
    a.tiny = 1e-14 * (fabs(bias) + 1.0);
    a.bias = bias;
    a.top = (double)((1u << bits) - 1u);
    a.seed = seed;
    a.fidx = fidx;
    a.nx = nx;
    a.ny = ny;
    if (f64)
        launch_t((const double *)frame, prnu, a, shot, adu, s);
    else
        launch_t((const float *)frame, prnu, a, shot, adu, s);
    return hipGetLastError();
}

}  // namespace e2e
