// Photon noise on the final frame (Sec. 2.2): every pixel's expected count
// becomes a Poisson draw.  Uniforms come from Philox-4x32-10 (Salmon,
// Moraes, Dror, Shaw, SC'11) with key = seed and counter = (pixel lo, pixel
// hi, frame index, draw block), so a pixel's draws depend only on
// (seed, frame, pixel): identical alone or inside any batch.  Means below 10
// use Knuth's multiplication method (TAOCP vol. 2, 3.4.1); larger means use
// Hormann's PTRS transformed rejection (Insurance: Math. & Econ. 12, 1993).
// A workgroup takes a span of up to 4096 pixels through poisson_span(), the
// frame read and (each pixel once) written in place.  Bound by the sampler's
// FP64 and integer arithmetic: on a 9216^2 FP32 frame whose means are all
// above 10, 2.78 -> 1.29 ms (the same counts bit for bit).
#include "philox.h"

namespace e2e {

namespace {

constexpr int kSpan = 4096;  // pixels of a workgroup's lists

template <typename T>
__device__ __forceinline__ void noise_spans(T *frame, int64_t n, int span, uint64_t seed,
                                            uint32_t fidx, PoissonLists<kSpan> &L)
{
    for (int64_t base = (int64_t)blockIdx.x * span; base < n; base += (int64_t)gridDim.x * span) {
        T *f = frame + base;
        poisson_span<kSpan>(
            (int)(n - base < span ? n - base : span), seed, fidx,
            [&](int c) { return (double)f[c]; }, [&](int c) { return (uint64_t)(base + c); },
            [&](int c, double k) { f[c] = (T)k; }, L);
        __syncthreads();  // the lists are free again
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_noise(T *frame, int64_t n, int span, uint64_t seed,
                                               uint32_t fidx)
{
    __shared__ PoissonLists<kSpan> L;
    noise_spans(frame, n, span, seed, fidx, L);
}

__global__ __launch_bounds__(256) void k_noise_frames(const FrameDev *__restrict__ frames, int span)
{
    __shared__ PoissonLists<kSpan> L;
    const FrameDev &F = frames[blockIdx.y];
    if (!F.poisson) return;
    const int64_t n = (int64_t)F.nx * F.ny;
    if (F.out_f64) noise_spans((double *)F.out, n, span, F.seed, F.frame_index, L);
    else noise_spans((float *)F.out, n, span, F.seed, F.frame_index, L);
}

// Small frames: one thread per pixel, all its trials in one loop (no lists, no
// barriers).  Below 2^17 pixels the lists' few turns cost more than they pack:
// 256^2 13.5 us against 15.9, 512^2 21.8 against 19.5.
constexpr int64_t kEachPixel = 1 << 17;

template <typename T>
__global__ __launch_bounds__(256) void k_noise_each(T *frame, int64_t n, uint64_t seed, uint32_t fidx)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    Stream st = make_stream(seed, fidx, (uint64_t)p);
    frame[p] = (T)poisson((double)frame[p], st);
}

// Pixels a workgroup takes at a time: long spans keep the later trials dense,
// short ones spread a frame over the GPU (2048 workgroups at the least).
int span_of(int64_t n)
{
    int span = kSpan;
    while (span > 512 && n / span < 2048) span /= 2;
    return span;
}

__global__ void k_philox(uint64_t seed, uint32_t frame, uint64_t pixel0, int64_t n,
                         uint32_t blocks, uint32_t *out)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * (int64_t)blocks) return;
    uint64_t p = pixel0 + (uint64_t)(i / blocks);
    uint32_t b = (uint32_t)(i % blocks);
    uint32_t x0 = (uint32_t)p, x1 = (uint32_t)(p >> 32), x2 = frame, x3 = b;
    philox10(x0, x1, x2, x3, (uint32_t)seed, (uint32_t)(seed >> 32));
    out[i * 4 + 0] = x0;
    out[i * 4 + 1] = x1;
    out[i * 4 + 2] = x2;
    out[i * 4 + 3] = x3;
}

}  // namespace

hipError_t launch_noise(void *frame, int f64, int64_t n, uint64_t seed, uint32_t frame_index,
                        hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n < kEachPixel) {
        const dim3 grid((unsigned)((n + 255) / 256));
        if (f64)
            hipLaunchKernelGGL(k_noise_each<double>, grid, dim3(256), 0, s, (double *)frame, n, seed,
                               frame_index);
        else
            hipLaunchKernelGGL(k_noise_each<float>, grid, dim3(256), 0, s, (float *)frame, n, seed,
                               frame_index);
        return hipGetLastError();
    }
    const int span = span_of(n);
    const int64_t nb64 = (n + span - 1) / span;
    const int nb = (int)(nb64 < 65536 ? nb64 : 65536);
    if (f64)
        hipLaunchKernelGGL(k_noise<double>, dim3(nb), dim3(256), 0, s, (double *)frame, n, span,
                           seed, frame_index);
    else
        hipLaunchKernelGGL(k_noise<float>, dim3(nb), dim3(256), 0, s, (float *)frame, n, span, seed,
                           frame_index);
    return hipGetLastError();
}

hipError_t launch_noise_frames(const FrameDev *frames_dev, const FrameDev *frames_host,
                               int n_frames, hipStream_t s)
{
    int64_t maxn = 0;
    bool any = false;
    for (int f = 0; f < n_frames; ++f) {
        if (!frames_host[f].poisson) continue;
        any = true;
        int64_t n = (int64_t)frames_host[f].nx * frames_host[f].ny;
        if (n > maxn) maxn = n;
    }
    if (!any) return hipSuccess;
    const int span = span_of(maxn);
    const int64_t nb64 = (maxn + span - 1) / span;
    const int nb = (int)(nb64 < 32768 ? nb64 : 32768);
    hipLaunchKernelGGL(k_noise_frames, dim3(nb, n_frames), dim3(256), 0, s, frames_dev, span);
    return hipGetLastError();
}

hipError_t launch_philox(uint64_t seed, uint32_t frame, uint64_t pixel0, int64_t n,
                         uint32_t blocks, uint32_t *out, hipStream_t s)
{
    int64_t tot = n * (int64_t)blocks;
    if (tot <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_philox, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, seed,
                       frame, pixel0, n, blocks, out);
    return hipGetLastError();
}

}  // namespace e2e
