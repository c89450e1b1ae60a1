// Closing the loop from the frame back to a radial velocity (Sec. 1: the
// simulated frames feed a data-reduction pipeline; Sec. 4.2: 1-D spectra
// extracted along the traced orders, the wavelength scale from the
// dispersion, the RV recovered by cross-correlation).
//
//  * k_extract: one thread per (trace, pixel column edge): the format
//    coordinate of the edge and of the column centre by safeguarded Newton
//    on x(t) (FP64), the edge wavelength, and the column's box extraction
//    over the rows within +-A of the trace centre (fractional end rows).
//    Neighbouring lanes read neighbouring pixels of each row.
//  * k_smooth3 / k_box_pass: the three passes of a clipped moving mean over a
//    template (the input spectrum of a trace): all three in one launch while
//    the window is narrow, from registers and one LDS array of prefix sums,
//    else one launch per pass.  Traces that share a template and a width (the
//    slices of a fiber) share its smoothed copy.
//  * k_ccf_mean / k_ccf / k_ccf_sum (k_ccf_runs and k_ccf_total): the mean of the flat-divided flux over
//    the usable columns; then a workgroup per (trace, run of columns) stages
//    the stretch of the smoothed template that a few columns read under every
//    trial velocity in LDS and adds up all velocities from there (linear
//    interpolation at the Doppler-shifted column centre); fixed-order sums
//    over the workgroups, and over the traces.
#include "dev_common.h"

namespace e2e {

namespace {

// Format coordinate t in [-1, 1] with x(t) = xe, x increasing on [-1, 1]
// (xa = x(-1) <= xe <= xb = x(1)): Newton steps from the linear guess,
// kept inside the shrinking bracket (bisection when a step would leave it).
__device__ double t_at_x(const double *cx, double xe, double xa, double xb)
{
    double lo = -1.0, hi = 1.0;
    double t = xb > xa ? fma(2.0, (xe - xa) / (xb - xa), -1.0) : 0.0;
    t = fmin(fmax(t, lo), hi);
    for (int it = 0; it < 64; ++it) {
        double d;
        const double f = horner_d<kNCoef - 1>(cx, t, &d) - xe;
        if (f == 0.0) break;
        if (f < 0.0) lo = t;
        else hi = t;
        double tn = d > 0.0 ? t - f / d : 0.5 * (lo + hi);
        if (!(tn > lo && tn < hi)) tn = 0.5 * (lo + hi);
        if (tn == t || hi - lo <= 0.0) break;
        t = tn;
    }
    return t;
}

template <typename T>
__global__ __launch_bounds__(256) void k_extract(const TraceDev *__restrict__ trs, int nx, int ny,
                                                 const T *__restrict__ frame, double A,
                                                 double *__restrict__ flux,
                                                 double *__restrict__ edges)
{
    const int e = blockIdx.x * 256 + threadIdx.x, tr = blockIdx.y;
    if (e > nx) return;
    const TraceDev &Tr = trs[tr];
    const double xa = horner<kNCoef - 1>(Tr.cx, -1.0), xb = horner<kNCoef - 1>(Tr.cx, 1.0);
    const double span = Tr.lmax - Tr.lmin;
    const double xe = (double)e - 0.5;
    double lam = __builtin_nan("");
    if (xe >= xa && xe <= xb) {
        const double t = t_at_x(Tr.cx, xe, xa, xb);
        lam = 0.5 * fma(t, span, Tr.lmin + Tr.lmax);
    }
    edges[(size_t)tr * (nx + 1) + e] = lam;
    if (e == nx) return;
    const int i = e;
    double acc = 0.0;
    if ((double)i - 0.5 >= xa && (double)i + 0.5 <= xb) {
        const double yc = horner<kNCoef - 1>(Tr.cy, t_at_x(Tr.cx, (double)i, xa, xb));
        const double lo = yc - A, hi = yc + A;
        const int j0 = max(0, (int)floor(lo + 0.5)), j1 = min(ny - 1, (int)floor(hi + 0.5));
        for (int j = j0; j <= j1; ++j) {
            const double ov = fmin((double)j + 0.5, hi) - fmax((double)j - 0.5, lo);
            if (ov > 0.0) acc = fma(ov, (double)frame[(size_t)j * nx + i], acc);
        }
    }
    flux[(size_t)tr * nx + i] = acc;
}

// A template to smooth.
struct LoopTemplate {
    const void *tmpl;   // spectrum slot, FP32 or FP64
    double *P;          // between the passes of a wide window, n values
    double *X;          // smoothed template, n
    int64_t n;
    int32_t w;          // moving-mean width (odd)
    int32_t pad;
};

// A trace of the CCF: its number and its smoothed template's.
struct LoopTrace {
    int32_t trace, tmpl;
};

constexpr int SMT = 2048;        // smoothed samples per workgroup (one pass)
constexpr int SMW = 4095;        // widest moving mean

__device__ void lds_scan(double *q, int len, double *tsum)
{
    // q[1 .. len] -> inclusive prefix sums in place (q[0] = 0): each thread
    // sums a run of consecutive values, the run totals are scanned with wave
    // shuffles and the four wave totals (fixed order), then each thread
    // rewrites its run
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int r = (len + 255) / 256;
    const int a = 1 + tid * r, b = min(len + 1, a + r);
    double run = 0.0;
    for (int k = a; k < b; ++k) run += q[k];
    double x = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) tsum[wv] = x;
    __syncthreads();
    double off = x - run;
    for (int u = 0; u < wv; ++u) off += tsum[u];
    for (int k = a; k < b; ++k) {
        off += q[k];
        q[k] = off;
    }
    __syncthreads();
}

// One moving-mean pass over a tile of SMT outputs of one trace: the tile's
// inputs with a half-window on each side are staged in LDS, scanned (FP64),
// and each output is the window sum (the
// window clipped to the array) over its count.  Pass 0 reads the template
// into X, pass 1 X into P, pass 2 P into X.
template <typename TT>
__global__ __launch_bounds__(256) void k_box_pass(const LoopTemplate *__restrict__ lt, int pass)
{
    __shared__ double q[SMT + SMW + 1];
    __shared__ double tsum[4];
    const LoopTemplate L = lt[blockIdx.y];
    const int64_t n = L.n, h = L.w / 2;
    const int64_t t0 = (int64_t)blockIdx.x * SMT;
    if (t0 >= n) return;
    const int64_t t1 = t0 + SMT < n ? t0 + SMT : n;
    const int64_t base = t0 - h > 0 ? t0 - h : 0, end = t1 + h < n ? t1 + h : n;
    const int len = (int)(end - base);
    const double *src = pass == 1 ? L.X : L.P;
    double *dst = pass == 1 ? L.P : L.X;
    const int tid = threadIdx.x;
    for (int k = tid; k < len; k += 256)
        q[k + 1] = pass == 0 ? (double)((const TT *)L.tmpl)[base + k] : src[base + k];
    if (tid == 0) q[0] = 0.0;
    __syncthreads();
    lds_scan(q, len, tsum);
    for (int64_t i = t0 + tid; i < t1; i += 256) {
        const int64_t lo = i - h > 0 ? i - h : 0, hi = i + h + 1 < n ? i + h + 1 : n;
        dst[i] = (q[hi - base] - q[lo - base]) / (double)(hi - lo);
    }
}

// All three passes in one launch.  A workgroup covers SL consecutive samples,
// its outputs and 3h on each side (clipped to the template); each thread keeps
// a run of SR of them in registers through the passes.  A pass scans the runs
// (registers, wave shuffles, the four wave totals), writes the exclusive prefix
// sums to LDS, and takes each output as the difference of two of them; the
// range that holds valid values shrinks by h a side each time.  SR is odd, so
// the 64-bit reads and writes of a wave fall on distinct banks.  The version
// before this one scanned in LDS, a run of 12 values a thread (eight lanes to a
// bank) and divided every output: 64 templates of 1e6 samples, w = 279,
// 765 us; this one 0.34 ms for as many (2.3 TB/s).
constexpr int STH = 512, SR = 9, SL = STH * SR;
constexpr int SFH = 512;         // widest half-window: at least SL - 6 * 512 = 1536 outputs

template <typename TT>
__global__ __launch_bounds__(STH) void k_smooth3(const LoopTemplate *__restrict__ lt, int outs)
{
    __shared__ double q[SL + 1];
    __shared__ double tsum[STH / 64];
    const LoopTemplate L = lt[blockIdx.y];
    const int64_t n = L.n, h = L.w / 2;
    const int64_t t0 = (int64_t)blockIdx.x * outs;
    if (t0 >= n) return;
    const int64_t t1 = t0 + outs < n ? t0 + outs : n;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t b = t0 - 3 * h > 0 ? t0 - 3 * h : 0, e = t1 + 3 * h < n ? t1 + 3 * h : n;
    const int len = (int)(e - b);
    for (int k = tid; k < SL; k += STH) q[k] = k < len ? (double)((const TT *)L.tmpl)[b + k] : 0.0;
    __syncthreads();
    double v[SR];
    const int i0 = tid * SR;
#pragma unroll
    for (int j = 0; j < SR; ++j) v[j] = q[i0 + j];
    const bool clipped = t0 < 3 * h || t1 + 3 * h > n;
    const double inv = 1.0 / (double)(2 * h + 1);
    const int hh = (int)h;
    for (int pass = 1; pass <= 3; ++pass) {
        double run = 0.0;
#pragma unroll
        for (int j = 0; j < SR; ++j) run += v[j];
        double x = run;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const double y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == 63) tsum[wv] = x;
        __syncthreads();  // also: every wave has read its values of the last pass
        double off = x - run;
        for (int u = 0; u < wv; ++u) off += tsum[u];
#pragma unroll
        for (int j = 0; j < SR; ++j) {
            q[i0 + j] = off;
            off += v[j];
        }
        if (tid == STH - 1) q[SL] = off;
        __syncthreads();
        // this pass's outputs lie in [lo, hi) of the workgroup's range
        const int64_t wb = (int64_t)(3 - pass) * h;
        const int lo = (int)((t0 - wb > 0 ? t0 - wb : 0) - b);
        const int hi = (int)((t1 + wb < n ? t1 + wb : n) - b);
        if (!clipped) {
#pragma unroll
            for (int j = 0; j < SR; ++j) {
                const int i = i0 + j;
                v[j] = i >= lo && i < hi ? (q[i + hh + 1] - q[i - hh]) * inv : 0.0;
            }
        } else {
#pragma unroll
            for (int j = 0; j < SR; ++j) {
                const int i = i0 + j;
                v[j] = 0.0;
                if (i >= lo && i < hi) {
                    const int64_t g = b + i;
                    const int64_t ga = g - h > 0 ? g - h : 0, gb = g + h + 1 < n ? g + h + 1 : n;
                    v[j] = (q[gb - b] - q[ga - b]) / (double)(gb - ga);
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < SR; ++j) q[i0 + j] = v[j];
    __syncthreads();
    for (int64_t i = t0 + tid; i < t1; i += STH) L.X[i] = q[i - b];
}

// The columns that enter a trace's CCF, and where its template is read.
struct CcfTrace {
    const double *F, *Ff, *Lt;
    double lmin, inv_dl, dmin, dmax, gmin, gmax, ulo, uhi;
    __device__ CcfTrace(const TraceDev &Tr, const LoopTemplate &L, int tr, int nx, const double *flux,
                        const double *flat, const double *edges, double v0, double dv, int nv)
    {
        const double c = 299792458.0;
        const double va = v0, vb = v0 + (nv - 1) * dv;
        F = flux + (size_t)tr * nx;
        Ff = flat ? flat + (size_t)tr * nx : nullptr;
        Lt = edges + (size_t)tr * (nx + 1);
        lmin = Tr.lmin;
        inv_dl = (double)L.n / (Tr.lmax - Tr.lmin);
        dmax = 1.0 + fmax(va, vb) / c;
        dmin = 1.0 + fmin(va, vb) / c;
        gmin = 1.0 / dmax;
        gmax = 1.0 / dmin;
        const int h = L.w / 2;
        ulo = 6.0 * h;
        uhi = (double)(L.n - 2 - 6 * h);
    }
    // fractional sample read at column centre lc under the factor d = 1 + v / c,
    // g = 1 / d (the quotient lc / d rounded as a division's: an error in it is
    // common to all columns of a velocity)
    __device__ double sample(double lc, double d, double g) const
    {
        const double q = lc * g;
        return fma(fma(fma(-q, d, lc), g, q) - lmin, inv_dl, -0.5);
    }
    __device__ double first(double lc) const { return sample(lc, dmax, gmin); }
    __device__ double last(double lc) const { return sample(lc, dmin, gmax); }
    __device__ bool usable(int i, double *lc, double *e) const
    {
        const double a = Lt[i], b = Lt[i + 1];
        if (isnan(a) || isnan(b)) return false;
        if (Ff && !(Ff[i] > 0.0)) return false;
        *lc = 0.5 * (a + b);
        *e = Ff ? F[i] / Ff[i] : F[i];
        return first(*lc) >= ulo && last(*lc) <= uhi;
    }
};

// Mean of e over a trace's usable columns, one workgroup a trace.
__global__ __launch_bounds__(256) void k_ccf_mean(const TraceDev *__restrict__ trs,
                                                  const LoopTrace *__restrict__ tl,
                                                  const LoopTemplate *__restrict__ lt, int nx,
                                                  const double *__restrict__ flux,
                                                  const double *__restrict__ flat,
                                                  const double *__restrict__ edges, double v0,
                                                  double dv, int nv, double *__restrict__ mean)
{
    __shared__ double red[2][256];
    const int tid = threadIdx.x, tr = tl[blockIdx.x].trace;
    const CcfTrace T(trs[tr], lt[tl[blockIdx.x].tmpl], tr, nx, flux, flat, edges, v0, dv, nv);
    double s = 0.0, cnt = 0.0;
    for (int i = tid; i < nx; i += 256) {
        double lc, e;
        if (T.usable(i, &lc, &e)) {
            s += e;
            cnt += 1.0;
        }
    }
    red[0][tid] = s;
    red[1][tid] = cnt;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) {
            red[0][tid] += red[0][tid + o];
            red[1][tid] += red[1][tid + o];
        }
        __syncthreads();
    }
    if (tid == 0) mean[tr] = red[1][0] > 0.0 ? red[0][0] / red[1][0] : 0.0;
}

// CCF of a run of KR columns of one trace.  Neighbouring columns read stretches
// of the template that overlap in most of their length (101 velocities span
// 2500 samples of a C1-shaped template, columns are 108 apart), so the columns
// go in steps whose stretch fits LDS, staged by coalesced loads; every
// (column, velocity) pair then reads its two samples from LDS.  (Read from
// global memory by a workgroup per 8 velocities, every load of a wave touched
// 64 lines and the template went through the caches 13 times: 833 us for 64
// traces, 265 us so.)  A step whose stretch does not fit (wide velocity grids
// on dense templates) reads global memory.
constexpr int KT = 512;          // threads
constexpr int KR = 512;          // columns per workgroup, at most
constexpr int KS = 64;           // columns per step, at most
constexpr int KX = 8960;         // template samples in LDS (two workgroups per CU)

__global__ __launch_bounds__(KT) void k_ccf(const TraceDev *__restrict__ trs,
                                            const LoopTrace *__restrict__ tl,
                                            const LoopTemplate *__restrict__ lt, int nx, int run,
                                            int step, const double *__restrict__ flux,
                                            const double *__restrict__ flat,
                                            const double *__restrict__ edges, double v0, double dv,
                                            int nv, int k0, int kn_all, int by_trace,
                                            const double *__restrict__ mean,
                                            double *__restrict__ part)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(16))) double sx[KX];
    __shared__ double slc[KR], se[KR];   // column centre (NaN: not used), e - mean
    const int tid = threadIdx.x, lane = tid & 63;
    const LoopTrace me = tl[blockIdx.y];
    const LoopTemplate L = lt[me.tmpl];
    const CcfTrace T(trs[me.trace], L, me.trace, nx, flux, flat, edges, v0, dv, nv);
    const double m0 = mean[me.trace];
    const int c_beg = blockIdx.x * run, cols = min(nx - c_beg, run);
    for (int c = tid; c < cols; c += KT) {
        double lc, e;
        const bool ok = T.usable(c_beg + c, &lc, &e);
        slc[c] = ok ? lc : __builtin_nan("");
        se[c] = ok ? e - m0 : 0.0;
    }
    __syncthreads();
    // threads share the velocities of a turn of up to KT: `ways` threads a
    // velocity, each every ways-th column
    double *const out =
        part + ((size_t)(by_trace ? me.trace : (int)blockIdx.y) * gridDim.x + blockIdx.x) * kn_all;
    for (int kb = 0; kb < kn_all; kb += KT) {
        const int kn = min(KT, kn_all - kb), ways = KT / kn;
        const int k = k0 + kb + tid % kn, way = tid / kn;
        const double d = 1.0 + (v0 + k * dv) / 299792458.0, g = 1.0 / d;
        double acc = 0.0;
        for (int c0 = 0; c0 < cols; c0 += step) {
            const int cn = min(step, cols - c0);
            // the stretch that the step's columns read (each wave finds it)
            const double mine = lane < cn ? slc[c0 + lane] : __builtin_nan("");
            double lo = isnan(mine) ? 1e300 : T.first(mine), hi = isnan(mine) ? -1e300 : T.last(mine);
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                lo = fmin(lo, __shfl_xor(lo, o));
                hi = fmax(hi, __shfl_xor(hi, o));
            }
            lo = uniform_d(lo);
            hi = uniform_d(hi);
            if (lo > hi) continue;  // no column used (the same in every wave)
            const int64_t xa = (int64_t)floor(lo) - 1, xb = (int64_t)floor(hi) + 3;
            const int64_t ra = (xa > 0 ? xa : 0) & ~(int64_t)1, rb = xb < L.n ? xb : L.n;
            const bool fits = rb - ra <= KX;
            if (fits) {
                const int len = (int)(rb - ra);
                const double *src = L.X + ra;   // 16-byte aligned: ra and the templates' spacing are even
                for (int q = 2 * tid; q + 1 < len; q += 2 * KT)
                    *reinterpret_cast<d2 *>(sx + q) = *reinterpret_cast<const d2 *>(src + q);
                if ((len & 1) && tid == 0) sx[len - 1] = src[len - 1];
                __syncthreads();
            }
            if (way < ways) {
                for (int j = way; j < cn; j += ways) {
                    const double lc = slc[c0 + j];
                    if (isnan(lc)) continue;
                    const double u = T.sample(lc, d, g), fl = floor(u);
                    const double f = u - fl;
                    double a, b;
                    if (fits) {
                        const double *p = sx + ((int64_t)fl - ra);
                        a = p[0];
                        b = p[1];
                    } else {
                        const double *p = L.X + (int64_t)fl;
                        a = p[0];
                        b = p[1];
                    }
                    acc = fma(se[c0 + j], fma(b - a, f, a), acc);
                }
            }
            __syncthreads();
        }
        double *const red = sx;   // free between the turns
        red[tid] = acc;
        __syncthreads();
        if (tid < kn) {
            double s = 0.0;
            for (int w = 0; w < ways; ++w) s += red[w * kn + tid];
            out[kb + tid] = s;
        }
        __syncthreads();
    }
}

// One workgroup a velocity: ccf[tr][k], the trace's column runs added in order,
// and their sum over the traces (each thread's in order, then the threads').
__global__ __launch_bounds__(256) void k_ccf_sum(const double *__restrict__ part, int runs, int ntr,
                                                 int nv, double *__restrict__ C,
                                                 double *__restrict__ tot)
{
    __shared__ double red[256];
    const int k = blockIdx.x, tid = threadIdx.x;
    double all = 0.0;
    for (int t = tid; t < ntr; t += 256) {
        const double *p = part + (size_t)t * runs * nv + k;
        double s = 0.0;
        for (int r = 0; r < runs; ++r) s += p[(size_t)r * nv];
        C[(size_t)t * nv + k] = s;
        all += s;
    }
    red[tid] = all;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) red[tid] += red[tid + o];
        __syncthreads();
    }
    if (tid == 0) tot[k] = red[0];
}

// The same in two kernels, where the partial sums of all traces and velocities are
// too many to hold: ccf[tr][k0 + k] of a launch's traces and velocities,
__global__ __launch_bounds__(256) void k_ccf_runs(const double *__restrict__ part,
                                                  const LoopTrace *__restrict__ tl, int runs, int nv,
                                                  int k0, int kn, double *__restrict__ C)
{
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= kn) return;
    const double *p = part + (size_t)blockIdx.y * runs * kn + k;
    double s = 0.0;
    for (int r = 0; r < runs; ++r) s += p[(size_t)r * kn];
    C[(size_t)tl[blockIdx.y].trace * nv + k0 + k] = s;
}

// and at the end the sum over the traces.
__global__ __launch_bounds__(256) void k_ccf_total(const double *__restrict__ C, int ntr, int nv, int k0,
                                                   double *__restrict__ tot)
{
    __shared__ double red[256];
    const int k = k0 + blockIdx.x, tid = threadIdx.x;
    double all = 0.0;
    for (int t = tid; t < ntr; t += 256) all += C[(size_t)t * nv + k];
    red[tid] = all;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (tid < o) red[tid] += red[tid + o];
        __syncthreads();
    }
    if (tid == 0) tot[k] = red[0];
}

}  // namespace

hipError_t launch_extract(const TraceDev *trs, int ntr, int nx, int ny, const void *frame,
                          int f64, double A, double *flux, double *edges, hipStream_t s)
{
    if (ntr <= 0 || nx <= 0) return hipSuccess;
    const dim3 grid((nx + 1 + 255) / 256, ntr);
    if (f64)
        hipLaunchKernelGGL(k_extract<double>, grid, dim3(256), 0, s, trs, nx, ny,
                           (const double *)frame, A, flux, edges);
    else
        hipLaunchKernelGGL(k_extract<float>, grid, dim3(256), 0, s, trs, nx, ny,
                           (const float *)frame, A, flux, edges);
    return hipGetLastError();
}

bool loop_needs_p(int w);
constexpr int kGridY = 65535;   // workgroups of a launch's second dimension
int loop_max_templates() { return kGridY; }

// (n_tmpl at most loop_max_templates())
hipError_t launch_smooth3(const void *lt_dev, int n_tmpl, int64_t nmax, int wmax, int f64,
                          hipStream_t s)
{
    if (n_tmpl <= 0 || nmax <= 0) return hipSuccess;
    const LoopTemplate *lt = (const LoopTemplate *)lt_dev;
    if (!loop_needs_p(wmax)) {
        const int outs = SL - 6 * (wmax / 2);
        const dim3 grid((unsigned)((nmax + outs - 1) / outs), n_tmpl);
        if (f64) hipLaunchKernelGGL(k_smooth3<double>, grid, dim3(STH), 0, s, lt, outs);
        else hipLaunchKernelGGL(k_smooth3<float>, grid, dim3(STH), 0, s, lt, outs);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((nmax + SMT - 1) / SMT), n_tmpl);
    for (int pass = 0; pass < 3; ++pass) {
        if (f64) hipLaunchKernelGGL(k_box_pass<double>, grid, dim3(256), 0, s, lt, pass);
        else hipLaunchKernelGGL(k_box_pass<float>, grid, dim3(256), 0, s, lt, pass);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

int loop_max_width() { return SMW; }
bool loop_needs_p(int w) { return w / 2 > SFH; }
// Columns a workgroup takes: 512, fewer while the launch would leave CUs idle.
static int ccf_run(int nx, int ntr)
{
    int run = KR;
    while (run > KS && (int64_t)ntr * ((nx + run - 1) / run) < 1024) run /= 2;
    return run;
}
int ccf_runs(int nx, int ntr) { return (nx + ccf_run(nx, ntr) - 1) / ccf_run(nx, ntr); }

hipError_t launch_ccf_mean(const TraceDev *trs, const void *tl_dev, int n_tr, const void *lt_dev,
                           int nx, const double *flux, const double *flat, const double *edges,
                           double v0, double dv, int nv, double *mean, hipStream_t s)
{
    if (n_tr <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ccf_mean, dim3(n_tr), dim3(256), 0, s, trs, (const LoopTrace *)tl_dev,
                       (const LoopTemplate *)lt_dev, nx, flux, flat, edges, v0, dv, nv, mean);
    return hipGetLastError();
}

// Partial sums at a time (bytes), and the velocities of a launch: longer grids go
// slice by slice (whole turns of KT: a velocity's sum is the same in any slice).
// Where the sums of all traces fit, one kernel at the end adds them up (with eight
// groups of templates 2.56 ms against 2.61 for a kernel after each group).
constexpr size_t kCcfPart = (size_t)128 << 20;
constexpr int kCcfSlice = 8 * KT;
static size_t ccf_trace_bytes(int nx, int ntr, int nv)
{
    return (size_t)ccf_runs(nx, ntr) * (nv < kCcfSlice ? nv : kCcfSlice) * sizeof(double);
}
static int ccf_traces(int nx, int ntr, int nv)   // of a launch
{
    const size_t fit = kCcfPart / ccf_trace_bytes(nx, ntr, nv);
    return (int)(fit < 1 ? 1 : fit < (size_t)kGridY ? fit : (size_t)kGridY);
}
static bool ccf_whole(int nx, int ntr, int nv) { return nv <= kCcfSlice && ntr <= ccf_traces(nx, ntr, nv); }
size_t ccf_part_bytes(int nx, int ntr, int nv)
{
    const int most = ccf_traces(nx, ntr, nv);
    return (ntr < most ? ntr : most) * ccf_trace_bytes(nx, ntr, nv);
}

// n_tr of the format's ntr traces, their partial sums or their rows of C (see
// ccf_whole); step: columns whose reads are
// expected to fit LDS, for templates of at most `spp` samples a column and a
// velocity grid of `vspan` samples
hipError_t launch_ccf(const TraceDev *trs, const void *tl_dev, int n_tr, int ntr, const void *lt_dev,
                      int nx, double spp, double vspan, const double *flux, const double *flat,
                      const double *edges, double v0, double dv, int nv, const double *mean,
                      double *part, double *C, hipStream_t s)
{
    const double fit = (KX - 8 - vspan) / (spp > 1e-6 ? spp : 1e-6);
    const int step = fit >= KS ? KS : fit >= 4.0 ? (int)fit : KS;
    const int runs = ccf_runs(nx, ntr), most = ccf_traces(nx, ntr, nv);
    const bool whole = ccf_whole(nx, ntr, nv);
    for (int t = 0; t < n_tr; t += most) {
        const int n = n_tr - t < most ? n_tr - t : most;
        const LoopTrace *tl = (const LoopTrace *)tl_dev + t;
        for (int k0 = 0; k0 < nv;) {
            const int kn = nv - k0 < kCcfSlice ? nv - k0 : kCcfSlice;
            hipLaunchKernelGGL(k_ccf, dim3(runs, n), dim3(KT), 0, s, trs, tl, (const LoopTemplate *)lt_dev,
                               nx, ccf_run(nx, ntr), step, flux, flat, edges, v0, dv, nv, k0, kn, (int)whole, mean,
                               part);
            if (!whole)
                hipLaunchKernelGGL(k_ccf_runs, dim3((kn + 255) / 256, n), dim3(256), 0, s, part, tl, runs,
                                   nv, k0, kn, C);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            k0 += kn;
        }
    }
    return hipSuccess;
}

hipError_t launch_ccf_total(const double *part, int ntr, int nx, int nv, double *C, double *tot,
                            hipStream_t s)
{
    if (ccf_whole(nx, ntr, nv)) {
        hipLaunchKernelGGL(k_ccf_sum, dim3(nv), dim3(256), 0, s, part, ccf_runs(nx, ntr), ntr, nv, C, tot);
        return hipGetLastError();
    }
    for (int k0 = 0; k0 < nv;) {
        const int kn = nv - k0 < (1 << 20) ? nv - k0 : 1 << 20;
        hipLaunchKernelGGL(k_ccf_total, dim3(kn), dim3(256), 0, s, C, ntr, nv, k0, tot);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        k0 += kn;
    }
    return hipSuccess;
}

size_t loop_template_bytes() { return sizeof(LoopTemplate); }
size_t loop_trace_bytes() { return sizeof(LoopTrace); }

void loop_template_fill(void *dst, const void *tmpl, double *P, double *X, int64_t n, int w)
{
    LoopTemplate L;
    L.tmpl = tmpl;
    L.P = P;
    L.X = X;
    L.n = n;
    L.w = w;
    L.pad = 0;
    *(LoopTemplate *)dst = L;
}

void loop_trace_fill(void *dst, int trace, int tmpl)
{
    LoopTrace L;
    L.trace = trace;
    L.tmpl = tmpl;
    *(LoopTrace *)dst = L;
}

}  // namespace e2e
