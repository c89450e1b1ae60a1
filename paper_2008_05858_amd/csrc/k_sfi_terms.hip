// Explicit spectral-fiber images of FP32 frames (Sec. 2.2), rendered as a
// product of their separable terms.
//
// With the fiber's chord points (a_p, h_p, w_p) of k_sfi.hip, a sample's
// weight on pixel (i, j) is a sum of R separable terms,
//     W(i, j) ~ sum_p X_p[i] Y_p[j],
//     X_p[i] = w_p (1/S) sum_s [N(u_is - a_p) + N(u_is + a_p)],
//     Y_p[j] = (1/S) sum_t [Phi~(v_jt - lo_p) - Phi~(v_jt - hi_p)],
// over the S sub-pixel centres of a pixel (N = exp(-z^2 / 2), Phi~ its
// integral).  k_sfi.hip evaluates the 2 R N S Gaussians and 2 R N S normal
// tails of a sample one by one (9.8 ms for 983,040 samples at S = 10, R = 9,
// N = 11 on 4096^2).  Here each mean over the sub-pixels is one expression,
// from the Taylor series in the sub-pixel offset u (moments m_2k = mean of
// u^2k, a function of S and sigma alone):
//     mean N(z + u)    = exp(-z^2/2) sum_k m_2k / (2k)! He_2k(z),
//     mean Phi~(z + u) = Phi~(z) - exp(-z^2/2) sum_k m_2k / (2k)! He_(2k-1)(z),
// polynomials in z^2 whose coefficients belong to the sample, with Phi~ from
// the Mills ratio (a fitted polynomial, relative error 1.2e-9).  Eight terms
// leave an error below 1e-9 of the peak for sigma >= 0.58 px (the rule in
// api.cpp; the terms fall as (1 / 2 sigma)^2k).  All in FP64, rounded once to
// FP32 operands.
//
// A workgroup owns a 64 x 32 tile.  Per chunk of up to 120 nodes, a node being
// one (sample, point) pair, one thread per (node, axis) walks the window once:
// it adds up its row (the window sum normalises the sample) and stores the
// in-tile entries in LDS in operand layout, as k_sep_fit.hip does; each
// sample's photons over its window sum scale its nodes where the products read
// them; wave w multiplies column block w, v_mfma_f32_16x16x4_f32, FP32 partials
// of eight nodes added to FP64 sums.  The order of every sum is fixed: the
// result is deterministic.
//
// Measured on that frame: 9.81 -> 1.84 ms (6.65 -> 1.85 at S = 1, 6.98 -> 1.88 at
// S = 2: the series do not grow with S, but even one sub-pixel centre costs the
// image-by-image form 2 R N Gaussians and tails); bound by VALU issue on the rows
// (the y rows twice the x rows).  Partials of 16 nodes took 1.78 ms and of four 2.01;
// on 2048^2 frames (S = 1 to 16) their largest error against 64 bits is 1.13e-7 to
// 1.22e-7 of the peak with 16, 0.94e-7 to 1.10e-7 with eight, 0.91e-7 to 1.05e-7 with
// four, image by image 1.18e-7 to 1.36e-7; of the norm 4.0e-8, 3.6e-8, 3.5e-8 and
// 4.5e-8 to 4.7e-8.
#include "sep_stage.h"

namespace e2e {

namespace {

constexpr int PB = 64;                   // samples positioned together
constexpr int K = 8;                     // terms of the sub-pixel series

// Mills ratio sqrt(2 pi) Phi(-z) exp(z^2 / 2), z >= 0 (fit_mills.py beside
// this file; relative error below 1.2e-9 up to z = 9, where exp(-z^2 / 2) is
// 1e-18)
__device__ __forceinline__ double mills(double z)
{
    const double v = fma(0.35, z, 1.0);
    double t = __builtin_amdgcn_rcp(v);
    t = fma(t, fma(-v, t, 1.0), t);
    double p = 4.54671504631161613e-02;
    p = fma(p, t, -3.29967897138510990e-01);
    p = fma(p, t, 9.95589412754607439e-01);
    p = fma(p, t, -1.54220537772396260e+00);
    p = fma(p, t, 1.21212149743348530e+00);
    p = fma(p, t, -5.44388352663080721e-01);
    p = fma(p, t, 4.59734635945394821e-01);
    p = fma(p, t, 2.48455457637747679e-01);
    p = fma(p, t, 3.59340801279976418e-01);
    p = fma(p, t, 3.49130936103494161e-01);
    return fma(p, t, 3.58727911046186065e-05);
}

// (-1/2)^m / m!
__device__ constexpr double kHalf[K + 1] = {
    1.0, -0.5, 0.125, -1.0 / 48.0, 1.0 / 384.0, -1.0 / 3840.0, 1.0 / 46080.0, -1.0 / 645120.0,
    1.0 / 10321920.0};
__device__ constexpr double kInvFact[2 * K + 1] = {
    1.0, 1.0, 1.0 / 2.0, 1.0 / 6.0, 1.0 / 24.0, 1.0 / 120.0, 1.0 / 720.0, 1.0 / 5040.0,
    1.0 / 40320.0, 1.0 / 362880.0, 1.0 / 3628800.0, 1.0 / 39916800.0, 1.0 / 479001600.0,
    1.0 / 6227020800.0, 1.0 / 87178291200.0, 1.0 / 1307674368000.0, 1.0 / 20922789888000.0};

template <int DX, int DY, typename ST>
__global__ __launch_bounds__(256, 3) void k_render_sfi_terms(const FrameDev *__restrict__ frames,
                                                             const int2 *__restrict__ work,
                                                             int n_work, int *__restrict__ counter,
                                                             int *__restrict__ err)
{
    constexpr int TX = kSfiTW, TY = kSfiTH;
    static_assert(TX == 64 && TY == 32 && CH == 120, "block geometry");
    __shared__ __attribute__((aligned(16))) float buf[(TX + TY) * LS];
    __shared__ __attribute__((aligned(16))) float sscl[LS];  // photons / window sum per node
    __shared__ double sxs[CH], sys[CH];      // window sums of a node's two rows
    __shared__ float sdx[PB], sdy[PB], ssx[PB], ssy[PB], sphi[PB];
    __shared__ int sax[PB], say[PB];         // first window column / row, relative to the tile
    __shared__ double smu[K + 1];            // mean of (2 u / pixel)^2k over the sub-pixel centres
    __shared__ float sfq[3 * kSfiMaxR];
    __shared__ unsigned short tlist[kMaxTileTraces];
    __shared__ unsigned smask[4][2];
    __shared__ unsigned long long sh_odd;    // samples whose photons are not ordinary numbers
    __shared__ int sh_item;
    float *const ybuf = buf + TX * LS;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int s = tid & 127;                 // staging role: node slot, axis (x: waves 0-1)
    const bool xaxis = tid < 128;

    for (int iter = 0;; ++iter) {
        int fi, tile_id;
        if (work == nullptr) {
            if (iter > 0) break;
            fi = 0;
            tile_id = xcd_remap(blockIdx.x, gridDim.x);
        } else {
            if (tid == 0) sh_item = atomicAdd(counter, 1);
            __syncthreads();
            const int w = uniform_i(sh_item);
            if (w >= n_work) break;
            const int2 wk = work[w];
            fi = uniform_i(wk.x);
            tile_id = uniform_i(wk.y);
        }
        const FrameDev &F = frames[fi];
        const int ntr = F.ntr, H = F.H, N = 2 * F.H + 1;
        const int R = F.sfi_R, S = F.sfi_S, shape = F.sfi_shape;
        const int tx = tile_id % F.ntx, ty = tile_id / F.ntx;
        const int X0 = tx * TX, Y0 = ty * TY;
        const SegDev *segs = F.segs + (size_t)tx * ntr;
        if (tid <= K) {
            double m = 0.0;
            for (int t = 0; t < S; ++t) {
                const double u = (double)(2 * t + 1) / (double)S - 1.0, u2 = u * u;
                double p = 1.0;
                for (int k = 0; k < tid; ++k) p *= u2;
                m += p;
            }
            smu[tid] = m / (double)S;
        }
        if (tid < 3 * R) sfq[tid] = F.sfq[tid];
        int count = tile_traces(segs, ntr, ty, tid, smask, tlist, err);
        zero_lines(buf, tid);
        if (tid < LS) sscl[tid] = 0.0f;
        __syncthreads();
        int zlo = 1, zhi = 0;  // lines this thread's node slot holds (none)
        double acc[2][4];
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[rb][q] = 0.0;

        for (int li = 0; li < count; ++li) {
            const int tr = uniform_i((int)tlist[li]);
            const TraceDev &T = F.tr[tr];
            const SegDev sg = segs[tr];
            double cxr[DX + 1], cyr[DY + 1];
#pragma unroll
            for (int j = 0; j <= DX; ++j) cxr[j] = T.cx[j];
#pragma unroll
            for (int j = 0; j <= DY; ++j) cyr[j] = T.cy[j];
            const TraceFrameDev &TF = F.tf[tr];
            const double t0 = TF.t0, dt = TF.dt;
            const double scale = TF.scale;
            const ST *spec = (const ST *)TF.spec;
            for (int kb = sg.k0; kb < sg.k1; kb += PB) {
                const int nb = min(PB, sg.k1 - kb);
                // 1. positions, windows, sigmas, photons of up to 64 samples
                bool odd = false;
                if (tid < nb) {
                    const int k = kb + tid;
                    const double t = fma((double)k, dt, t0);
                    const double x = horner<DX>(cxr, t);
                    const double y = horner<DY>(cyr, t);
                    const double axd = floor(x + 0.5), ayd = floor(y + 0.5);
                    float sgx, sgy;
                    sigma_at(F.sxy, F.gx, F.gy, F.gsx, F.gsy, x, y, &sgx, &sgy);
                    sdx[tid] = (float)(x - axd);
                    sdy[tid] = (float)(y - ayd);
                    ssx[tid] = sgx;
                    ssy[tid] = sgy;
                    sphi[tid] = (float)(spec_at(spec, k) * scale);
                    sax[tid] = (int)axd - H - X0;
                    say[tid] = (int)ayd - H - Y0;
                    odd = !(fabsf(sphi[tid]) < 1e30f);
                }
                {
                    static_assert(PB == 64, "the first wave holds them");
                    const unsigned long long m = __ballot(odd);
                    if (tid == 0) sh_odd = m;
                }
                __syncthreads();
                // chunks of equal length, each a whole number of samples
                const int most = CH / R, nch = (nb + most - 1) / most, per = (nb + nch - 1) / nch;
                for (int c0 = 0; c0 < nb; c0 += per) {
                    const int nk = min(per, nb - c0), nn = nk * R;
                    // 2. this thread's node and axis: its row over the window
                    {
                        int nlo = 1, nhi = 0;
                        const bool have = s < nn;
                        if (have) {
                            const int q = s / R, p = s - q * R, smp = c0 + q;
                            const double sg1 = (double)(xaxis ? ssx[smp] : ssy[smp]);
                            const double h = recip(sg1), a = 0.5 * h, a2 = a * a;
                            // b_k = m_2k: the mean of u^2k, u up to half a pixel
                            double b[K + 1], w = 1.0;
#pragma unroll
                            for (int k = 0; k <= K; ++k) {
                                b[k] = w * smu[k];
                                w *= a2;
                            }
                            const int off = xaxis ? sax[smp] : say[smp];
                            const int NL = xaxis ? TX : TY;
                            const double z0 = -((double)H + (double)(xaxis ? sdx[smp] : sdy[smp])) * h;
                            float *at = (xaxis ? buf : ybuf) + lds_at(off, s);
                            const double g0 = exp_mid(-h * h);
                            double tot = 0.0;
                            if (xaxis) {
                                const double al = (double)sfq[3 * p] * h, wp = (double)sfq[3 * p + 2];
                                // coefficients of sum_k b_k / (2k)! He_2k(z) in z^2
                                double C[K + 1];
#pragma unroll
                                for (int i = 0; i <= K; ++i) {
                                    double v = 0.0;
#pragma unroll
                                    for (int m = K - i; m >= 0; --m) v = fma(kHalf[m], b[i + m], v);
                                    C[i] = v * kInvFact[2 * i];
                                }
                                double za = z0 - al, zb = z0 + al;
                                double Ea = wp * exp_mid(-0.5 * za * za), Eb = wp * exp_mid(-0.5 * zb * zb);
                                double ra = exp_mid(-h * fma(0.5, h, za)), rb = exp_mid(-h * fma(0.5, h, zb));
                                for (int i = 0; i < N; ++i) {
                                    const double va = za * za, vb = zb * zb;
                                    double pa = C[K], pb = C[K];
#pragma unroll
                                    for (int k = K - 1; k >= 0; --k) {
                                        pa = fma(pa, va, C[k]);
                                        pb = fma(pb, vb, C[k]);
                                    }
                                    const double v = fma(Ea, pa, Eb * pb);
                                    tot += v;
                                    if ((unsigned)(off + i) < (unsigned)NL) at[0] = (float)v;
                                    at += LS;
                                    Ea *= ra;
                                    Eb *= rb;
                                    ra *= g0;
                                    rb *= g0;
                                    za += h;
                                    zb += h;
                                }
                                sxs[s] = tot;
                            } else {
                                const double hp = (double)sfq[3 * p + 1] * h;
                                const double e1 = shape == E2E_FIBER_HALF_UP ? 0.0 : hp;     // -lo
                                const double e2 = shape == E2E_FIBER_HALF_DOWN ? 0.0 : hp;   // hi
                                // coefficients of sum_k b_k / (2k)! He_(2k-1)(z) / z in z^2
                                double O[K];
#pragma unroll
                                for (int i = 0; i < K; ++i) {
                                    double v = 0.0;
#pragma unroll
                                    for (int m = K - 1 - i; m >= 0; --m)
                                        v = fma(kHalf[m] / (2.0 * (i + 1 + m)), b[i + 1 + m], v);
                                    O[i] = v * kInvFact[2 * i + 1];
                                }
                                double za = z0 + e1, zb = z0 - e2;
                                double Ea = exp_mid(-0.5 * za * za), Eb = exp_mid(-0.5 * zb * zb);
                                double ra = exp_mid(-h * fma(0.5, h, za)), rb = exp_mid(-h * fma(0.5, h, zb));
                                for (int j = 0; j < N; ++j) {
                                    // tails of the sub-pixel mean of Phi~ at |z|
                                    const double ua = fabs(za), ub = fabs(zb);
                                    const double va = za * za, vb = zb * zb;
                                    double pa = O[K - 1], pb = O[K - 1];
#pragma unroll
                                    for (int k = K - 2; k >= 0; --k) {
                                        pa = fma(pa, va, O[k]);
                                        pb = fma(pb, vb, O[k]);
                                    }
                                    const double ta = Ea * fma(pa, ua, mills(ua));
                                    const double tb = Eb * fma(pb, ub, mills(ub));
                                    // on the side where nothing cancels
                                    const double v = zb >= 0.0 ? tb - ta
                                                     : za <= 0.0 ? ta - tb
                                                                 : (2.5066282746310002 - ta) - tb;
                                    tot += v;
                                    if ((unsigned)(off + j) < (unsigned)NL) at[0] = (float)v;
                                    at += LS;
                                    Ea *= ra;
                                    Eb *= rb;
                                    ra *= g0;
                                    rb *= g0;
                                    za += h;
                                    zb += h;
                                }
                                sys[s] = tot;
                            }
                            nlo = max(off, 0);
                            nhi = min(off + N - 1, NL - 1);
                        }
                        if (nlo > nhi) nlo = 1, nhi = 0;
                        clear_lines(zlo, zhi, nlo, nhi, s, xaxis ? buf : ybuf);
                        zlo = nlo;
                        zhi = nhi;
                        group_masks(block_bits(nlo, nhi), lane, wv, smask);
                    }
                    __syncthreads();
                    // 3. each node's scale: the sample's photons over its window
                    // sum, sum_p (sum_i X_p[i]) (sum_j Y_p[j])
                    if (tid < CH) {
                        double z = 0.0;
                        const int q = tid / R;
                        if (tid < nn)
                            for (int p = 0; p < R; ++p)
                                z = fma(sxs[q * R + p], sys[q * R + p], z);
                        const bool use = tid < nn && !((sh_odd >> (c0 + q)) & 1u);
                        sscl[tid] = use ? (float)((double)sphi[c0 + q] * recip(z)) : 0.0f;
                    }
                    __syncthreads();
                    // 4. products
                    tile_products<true, 8>(buf, ybuf, sscl, smask, wv, l16, lg, acc);
                    // A NaN, an infinity (or a scale out of FP32's range) stays in
                    // its own window: the products would carry it to every pixel of
                    // its blocks of 16, so such a sample is added pixel by pixel.
                    if (__builtin_expect(uniform_i(sh_odd != 0), 0))
                        for (int q = 0; q < nk; ++q) {
                            const int smp = c0 + q;
                            if (!uniform_i((int)((sh_odd >> smp) & 1u))) continue;
                            double z = 0.0;
                            for (int p = 0; p < R; ++p)
                                z = fma(sxs[q * R + p], sys[q * R + p], z);
                            const double sc = (double)sphi[smp] / z;
                            const int col = 16 * wv + l16;
                            if ((unsigned)(col - sax[smp]) >= (unsigned)N) continue;
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const int row = 16 * (e >> 2) + 4 * lg + (e & 3);
                                if ((unsigned)(row - say[smp]) >= (unsigned)N) continue;
                                float v = 0.0f;
                                for (int p = 0; p < R; ++p)
                                    v = fmaf(buf[lds_at(col, q * R + p)], ybuf[lds_at(row, q * R + p)], v);
                                acc[e >> 2][e & 3] = fma((double)v, sc, acc[e >> 2][e & 3]);
                            }
                        }
                    __syncthreads();
                }
            }
        }
        put_tile(F, X0, Y0, wv, l16, lg, acc);
        __syncthreads();
    }
}

template <int DX, int DY>
hipError_t launch_deg(const FrameDev *frames_dev, const KernelCfg &cfg, const int2 *work,
                      int n_work, int *counter, int *err, int nb, hipStream_t s)
{
    if (cfg.spec_f64)
        hipLaunchKernelGGL((k_render_sfi_terms<DX, DY, double>), dim3(nb), dim3(256), 0, s,
                           frames_dev, work, n_work, counter, err);
    else
        hipLaunchKernelGGL((k_render_sfi_terms<DX, DY, float>), dim3(nb), dim3(256), 0, s,
                           frames_dev, work, n_work, counter, err);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_sfi_terms(const FrameDev *frames_dev, const KernelCfg &cfg, const int2 *work,
                            int n_work, int *counter, int *err, hipStream_t s)
{
    // plain: one workgroup per tile; persistent: three per CU
    const int nb = work == nullptr ? cfg.plain_tiles : (n_work < 768 ? n_work : 768);
    if (nb <= 0) return hipSuccess;
    if (cfg.degx <= 4 && cfg.degy <= 3)
        return launch_deg<4, 3>(frames_dev, cfg, work, n_work, counter, err, nb, s);
    return launch_deg<7, 7>(frames_dev, cfg, work, n_work, counter, err, nb, s);
}

}  // namespace e2e
