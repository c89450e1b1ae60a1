// Separable-PSF render path for FP32 frames (Sec. 2.1's axis-aligned
// Gaussian aberration model with field-dependent (sigma_x, sigma_y)): the
// samples of one trace in one pixel column are first gathered onto a few
// nodes, then the nodes are rendered.
//
// Within one pixel column of a trace (the samples with floor(x + 1/2) = i)
// and one row anchor, a sample's footprint is a smooth function of its place
// tau in [-1, 1] between the column's first and last sample: both windows
// stand still, and x, y, sigma_x and sigma_y vary smoothly along the trace.
// So the footprint is taken as its Chebyshev interpolant on the M nodes tau_m,
//     w(tau) = sum_m L_m(tau) w(tau_m),
// and the column's samples add up to M node weights
//     sum_k phi_k w(tau_k) = sum_m Phi_m w(tau_m),
//     Phi_m = sum_k phi_k L_m(tau_k) = 1/M (mu_0 + 2 sum_{p>=1} mu_p T_p(tau_m)),
//     mu_p = sum_k phi_k T_p(tau_k),
// FP64 sums over the samples by the recurrence of phi T_p.  For a Gaussian of
// inverse width kappa along the trace (x is linear in tau within the bend that
// sep_fit_nodes allows) the interpolation error is below
// 2.2 (kappa / 4)^M / sqrt(M!) of the footprint's peak (Cramer's bound on the
// Hermite functions): the host picks M = 10 or 12 so that this stays below
// 4e-9 (sep_fit_nodes), a tenth of the FP32 rounding of the frame.  Columns
// where the footprint is not smooth (a line of the sigma grid crosses them,
// the trace begins or ends in them) or that hold no more than M + 1 samples
// render their samples one by one.
//
// What bounds it: the C2-shaped frame (9216^2, 340 traces, 108 samples a
// column) used to evaluate 36 normal CDFs for each of 3.4e8 samples in every
// tile it reaches, VALU issue in all of the per-sample kernels.  Here a sample
// costs ~14 FP64 instructions (two mirrored samples share a recurrence; no
// position: nodes lie at sample numbers) and a tenth as many nodes the pixel
// integrals: 56.8 ms (FP64 VALU) -> 5.7 ms, 35.0 ms (fp16 hi/lo MFMA) -> 4.9 ms,
// still VALU issue, on the node's pixel integrals, the
// column sums and the FP64 additions of the products.  (With nodes at given x,
// found by Newton steps, and a position and a full recurrence for each sample
// it took 5.4 ms.)
//
// A workgroup owns a 64 x 32 tile, three of them fit a CU (LDS).  Per trace:
// the first sample of each column (exact test on the FP64 format), the column
// list, then for batches of columns: four lanes a column add up the moments
// and write the nodes' photons to LDS; then per chunk of 120 nodes one thread
// per (node, axis) stores the node's pixel integrals on the tile's 64 columns
// (times photons) or 32 rows as FP32, and finds the next chunk's position and
// sigma; wave w multiplies column block w, F += Gy diag(Phi) Gx^T, by
// v_mfma_f32_16x16x4_f32, FP32 partials of SPAN nodes added to FP64 sums: four
// under E2E_PREC_F64, 16 under the reduced precisions.  A pixel gathers about 30
// nodes, so a partial of 16 is half of it and its rounding shows: on frames of
// sigma 0.8 .. 1.6 px the largest error is 1.2e-7 to 1.7e-7 of the peak with 16
// (C2-shaped frame 4.89 ms), 0.9e-7 to 1.15e-7 with eight (5.17 ms) and 0.65e-7 to
// 0.99e-7 with four (5.73 ms), where FP64 sums of every sample leave 0.9e-7 to
// 1.4e-7 (56.4 ms), and the other precisions' per-sample forms 2e-7 (hi/lo) and
// 1e-6 to 2e-6 (FP32).  FP64 products (v_mfma_f64_16x16x4_f64) took 6.8 ms where
// 16 took 5.4, fp16 hi/lo halves 6.4 ms (splitting the weights costs more than the
// matrix cores save).
// Pixel integrals are taken in FP64: P(z) = 2a phi(z) sum_i A_i (z a)^(2i) /
// (2i)!, a = h / 2 = 1 / (2 sigma), from exp(-z u) expanded under the integral
// over the pixel (A_i = int_0^1 v^(2i) exp(-a^2 v^2 / 2) dv by its downward
// recurrence); the Gaussian runs along the window by two multiplications a
// pixel.  Eight terms leave an absolute error below 4e-10 for sigma >= 0.58.
// The order of every sum is fixed: the result is deterministic.
#include "sample_index.h"
#include "sep_stage.h"

namespace e2e {

namespace {

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int TX = kMfmaTW;            // 64 columns = 4 blocks of 16, one per wave
constexpr int TY = kMfmaTH;            // 32 rows = 2 blocks of 16
constexpr int NCOL = TX + 2 * kMaxH;   // pixel columns whose samples reach the tile
constexpr int NENT = 2 * NCOL;         // list entries: at most two row anchors a column

// the nodes tau_m = cos((2m + 1) pi / (2M))
__device__ constexpr double kNode10[10] = {
    0.98768834059513777, 0.8910065241883679, 0.70710678118654757, 0.4539904997395468,
    0.15643446504023092, -0.15643446504023092, -0.4539904997395468, -0.70710678118654757,
    -0.8910065241883679, -0.98768834059513777};
__device__ constexpr double kNode12[12] = {
    0.99144486137381038, 0.92387953251128674, 0.79335334029123517, 0.60876142900872066,
    0.38268343236508984, 0.13052619222005171, -0.13052619222005171, -0.38268343236508984,
    -0.60876142900872066, -0.79335334029123517, -0.92387953251128674, -0.99144486137381038};
// list entry: pixel column, row anchor (relative to the tile, + kMaxH), flags
constexpr unsigned kEntRaw = 1u << 14;   // samples one by one
constexpr unsigned kEntTest = 1u << 13;  // only the samples with this row anchor
__device__ __forceinline__ unsigned ent_pack(int col, int arow)
{
    return (unsigned)col | ((unsigned)(arow + kMaxH) << 7);
}

// Pixel integrals of one Gaussian (sigma sg, centre d from the anchor pixel)
// on NL pixel lines: window pixel m (0 .. 2H) lies on line off + m and gets
// its integral times scale / window sum.  Writes the in-tile entries and
// returns their line range (empty: *plo > *phi).
template <int NL>
__device__ __forceinline__ void stage_axis(double d, double sg, int H, double scale, int off,
                                           int s, float *b, int *plo, int *phi)
{
    const int m0 = max(0, -off), m1 = min(2 * H, NL - 1 - off);
    *plo = off + m0;
    *phi = off + m1;
    if (m0 > m1) return;
    const double h = recip(sg), a = 0.5 * h, a2 = a * a;
    const double e0 = exp_small(-0.5 * a2);
    // A_8 by its ascending series, then downward (all terms positive)
    double A = e0 * fma(a2, fma(a2, fma(a2, 1.0 / 156009.0, 1.0 / 6783.0), 1.0 / 323.0), 1.0 / 17.0);
    A = fma(a2, A, e0) * (1.0 / 15.0);
    const double c7 = A * (1.0 / 87178291200.0);
    A = fma(a2, A, e0) * (1.0 / 13.0);
    const double c6 = A * (1.0 / 479001600.0);
    A = fma(a2, A, e0) * (1.0 / 11.0);
    const double c5 = A * (1.0 / 3628800.0);
    A = fma(a2, A, e0) * (1.0 / 9.0);
    const double c4 = A * (1.0 / 40320.0);
    A = fma(a2, A, e0) * (1.0 / 7.0);
    const double c3 = A * (1.0 / 720.0);
    A = fma(a2, A, e0) * (1.0 / 5.0);
    const double c2 = A * (1.0 / 24.0);
    A = fma(a2, A, e0) * (1.0 / 3.0);
    const double c1 = A * 0.5;
    const double c0 = fma(a2, A, e0);
    // the window's outer edges lie in the far tail: the fitted FP32 tail's
    // relative error there is below 2e-7 of Phi(-H / sigma)
    const float ta = phi_tail_f32((float)(((double)(-H) - 0.5 - d) * h));
    const float tb = phi_tail_f32((float)(((double)H + 0.5 - d) * h));
    const double f = scale * 0.3989422804014327 * h * recip((1.0 - (double)ta) - (double)tb);
    double z = ((double)(m0 - H) - d) * h;
    double E = f * exp_mid(-0.5 * z * z), r = exp_mid(-h * fma(0.5, h, z));
    double q = e0 * e0;
    q *= q;
    q *= q;
    double w = z * a;
    const double dw = h * a;
    // two pixels a turn: two independent chains
    const double q2 = q * q, rq = r * r * q, dw2 = dw + dw;
    double E1 = E * r, w1 = w + dw;
    double g0 = rq, g1 = rq * q2;  // E_{m+2} / E_m, E_{m+3} / E_{m+1}
    float *at = b + lds_at(off + m0, s);
    const double q4 = q2 * q2;
    for (int m = m0; m <= m1; m += 2) {
        const double v0 = w * w, v1 = w1 * w1;
        double p0 = fma(c7, v0, c6), p1 = fma(c7, v1, c6);
        p0 = fma(p0, v0, c5);
        p1 = fma(p1, v1, c5);
        p0 = fma(p0, v0, c4);
        p1 = fma(p1, v1, c4);
        p0 = fma(p0, v0, c3);
        p1 = fma(p1, v1, c3);
        p0 = fma(p0, v0, c2);
        p1 = fma(p1, v1, c2);
        p0 = fma(p0, v0, c1);
        p1 = fma(p1, v1, c1);
        p0 = fma(p0, v0, c0);
        p1 = fma(p1, v1, c0);
        at[0] = (float)(E * p0);
        if (m < m1) at[LS] = (float)(E1 * p1);
        at += 2 * LS;
        E *= g0;
        E1 *= g1;
        g0 *= q4;
        g1 *= q4;
        w += dw2;
        w1 += dw2;
    }
}

// One axis' sigma of a sample, bilinear in the field over the node grid.
__device__ __forceinline__ double sigma_axis(const float *sxy, int gx, int gy, double gsx,
                                             double gsy, double x, double y, int c)
{
    double fx, fy;
    const int cx = node_cell(x, gsx, gx, &fx), cy = node_cell(y, gsy, gy, &fy);
    const int cx1 = min(cx + 1, gx - 1), cy1 = min(cy + 1, gy - 1);
    const float s00 = sxy[(cy * gx + cx) * 2 + c], s01 = sxy[(cy * gx + cx1) * 2 + c];
    const float s10 = sxy[(cy1 * gx + cx) * 2 + c], s11 = sxy[(cy1 * gx + cx1) * 2 + c];
    const double lo = fma(fx, (double)s01 - (double)s00, (double)s00);
    const double hi = fma(fx, (double)s11 - (double)s10, (double)s10);
    return fma(fy, hi - lo, lo);
}

// v added over the four lanes of a quad (the same bits in each)
__device__ __forceinline__ double quad_sum(double v)
{
    long long b = __double_as_longlong(v);
    int lo = (int)(b & 0xffffffffll), hi = (int)(b >> 32);
    int l1 = __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
    int h1 = __builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xF, 0xF, true);
    v += __longlong_as_double(((long long)h1 << 32) | (unsigned)l1);
    b = __double_as_longlong(v);
    lo = (int)(b & 0xffffffffll);
    hi = (int)(b >> 32);
    l1 = __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xF, 0xF, true);      // quad_perm [2,3,0,1]
    h1 = __builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xF, 0xF, true);
    return v + __longlong_as_double(((long long)h1 << 32) | (unsigned)l1);
}

template <typename ST>
struct Vec4;
template <>
struct Vec4<float> {
    __device__ static void load(const float *p, int k, float v[4])
    {
        const f4u q = *reinterpret_cast<const __attribute__((address_space(1))) f4u *>(as_global(p + k));
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    }
};
template <>
struct Vec4<double> {
    __device__ static void load(const double *p, int k, double v[4])
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = p[k + e];
    }
};

template <int DX, int DY, typename ST, int M, int SPAN, bool NARROW>
__global__ __launch_bounds__(256, 3) void k_render_sep_fit(const FrameDev *__restrict__ frames,
                                                           const int2 *__restrict__ work,
                                                           int n_work, int *__restrict__ counter,
                                                           int *__restrict__ err)
{
    constexpr int BE = M == 10 ? 60 : 50;   // list entries per batch (4 lanes each)
    static_assert(TX == 64 && TY == 32 && CH == 120, "block geometry");
    static_assert(NCOL <= 128 && TY + 2 * kMaxH < 64, "entry fields");
    __shared__ __attribute__((aligned(16))) float buf[(TX + TY) * LS];
    __shared__ float sphi[BE][M];           // node photons of the batch
    __shared__ int kst[NCOL + 1];           // first sample of each column
    __shared__ int noff[BE + 1];            // first node of each entry of the batch
    __shared__ unsigned short ent[NENT];
    __shared__ unsigned short tlist[kMaxTileTraces];
    __shared__ unsigned smask[4][2];
    __shared__ double snode[M];             // tau_m
    __shared__ int sh_item, sh_nent, sh_raw, sh_neg;
    float *const ybuf = buf + TX * LS;       // the rows' lines follow the columns'

    const int tid = threadIdx.x;
    if (tid < M) snode[tid] = M == 10 ? kNode10[tid % 10] : kNode12[tid];
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    // staging role: node slot s of the chunk, axis (x: waves 0-1, y: 2-3)
    const int s = tid & 127;
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
        const int ntr = F.ntr, H = F.H;
        const int tx = tile_id % F.ntx, ty = tile_id / F.ntx;
        const int X0 = tx * TX, Y0 = ty * TY;
        const int ncol = min(TX, F.nx - X0) + 2 * H;
        const SegDev *segs = F.segs + (size_t)tx * ntr;
        int count = tile_traces(segs, ntr, ty, tid, smask, tlist, err);
        zero_lines(buf, tid);
        if (NARROW && tid == 0) sh_neg = 0;
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
            const int nsamp = T.n;

            // ---- first sample of each pixel column X0 - H + c (the sample's
            // own test floor(x + 1/2) >= column), inside the planner's range
            if (tid <= ncol) {
                const int k0 = sg.k0, k1 = sg.k1;
                const double col = (double)(X0 - H + tid);
                auto xp = [&](int k) { return horner<DX>(cxr, fma((double)k, dt, t0)) + 0.5; };
                const int km = k0 + ((k1 - 1 - k0) >> 1);
                const double ua = xp(k0), um = xp(km), ub = xp(k1 - 1);
                int k;
                if (ua >= col) k = k0;
                else if (ub < col) k = k1;
                else {
                    // quadratic guess through three samples, then exact: the
                    // bracket [lo, hi] is widened from the guess and bisected
                    double d1 = (double)(k1 - 1 - k0) / (ub - ua), d2 = 0.0;
                    if (km > k0 && km < k1 - 1) {
                        d1 = (double)(km - k0) / (um - ua);
                        d2 = ((double)(k1 - 1 - km) / (ub - um) - d1) / (ub - ua);
                    }
                    const double g = ceil(fma(col - ua, fma(col - um, d2, d1), (double)k0));
                    k = min(max((int)fmin(fmax(g, (double)k0), (double)k1), k0 + 1), k1 - 1);
                    int lo = k0 + 1, hi = k1 - 1;  // the answer lies in [k0 + 1, k1 - 1]
                    if (xp(k) >= col) {
                        hi = k;
                        for (int step = 1; hi > lo; step *= 2) {
                            const int c = max(lo, hi - step);
                            if (xp(c) >= col) hi = c;
                            else { lo = c + 1; break; }
                        }
                    } else {
                        lo = k + 1;
                        for (int step = 1; lo < hi; step *= 2) {
                            const int c = hi - lo < step ? hi : lo + step - 1;
                            if (xp(c) < col) lo = c + 1;
                            else { hi = c; break; }
                        }
                    }
                    while (lo < hi) {
                        const int mid = lo + ((hi - lo) >> 1);
                        if (xp(mid) >= col) hi = mid; else lo = mid + 1;
                    }
                    k = lo;
                }
                kst[tid] = k;
            }
            __syncthreads();

            // ---- the columns that reach the tile's rows, one entry for each
            // row anchor (at most two, |dy/dx| <= 1/2), in column order
            if (wv == 0) {
                int n = 0;
                bool any_raw = false;
                for (int base = 0; base < ncol; base += 64) {
                    const int c = base + lane;
                    unsigned e0 = 0, e1 = 0;
                    int ne = 0;
                    if (c < ncol) {
                        const int ks = kst[c], ke = kst[c + 1];
                        if (ks < ke) {
                            const double ta = fma((double)ks, dt, t0);
                            const double tb = fma((double)(ke - 1), dt, t0);
                            const double ya = horner<DY>(cyr, ta), yb = horner<DY>(cyr, tb);
                            // |y - chord| <= y2max (tb - ta)^2 / 8
                            const double mg = fma(T.y2max, (tb - ta) * (tb - ta), 1e-9);
                            const double yl = fmin(ya, yb) - mg, yh = fmax(ya, yb) + mg;
                            const int al = (int)floor(yl + 0.5), ah = (int)floor(yh + 0.5);
                            if (ah + H >= Y0 && al - H < Y0 + TY) {
                                const double xc = (double)(X0 - H + c);
                                // a line of the sigma grid in the column (the
                                // nodes reach up to a sample past its ends in y)
                                const double ext = (yh - yl) / (double)max(ke - ks - 1, 1) + 1e-6;
                                const bool kink =
                                    ext_cell(xc - 0.500001, F.gsx, F.gx) !=
                                        ext_cell(xc + 0.500001, F.gsx, F.gx) ||
                                    ext_cell(yl - ext, F.gsy, F.gy) != ext_cell(yh + ext, F.gsy, F.gy);
                                const bool raw = ke - ks < M + 2 || ks == 0 || ke == nsamp || kink ||
                                                 ah > al + 1;
                                if (raw) {
                                    e0 = (unsigned)c | kEntRaw;
                                    ne = 1;
                                    any_raw = true;
                                } else {
                                    const bool two = al != ah;
                                    const bool in0 = al + H >= Y0 && al - H < Y0 + TY;
                                    const bool in1 = two && ah + H >= Y0 && ah - H < Y0 + TY;
                                    const unsigned tst = two ? kEntTest : 0u;
                                    const unsigned p0 = in0 ? ent_pack(c, al - Y0) | tst : 0u;
                                    const unsigned p1 = in1 ? ent_pack(c, ah - Y0) | tst : 0u;
                                    e0 = in0 ? p0 : p1;
                                    e1 = p1;
                                    ne = (in0 ? 1 : 0) + (in1 ? 1 : 0);
                                }
                            }
                        }
                    }
                    const unsigned long long b1 = __ballot(ne >= 1), b2 = __ballot(ne == 2);
                    const unsigned long long below = (1ull << lane) - 1ull;
                    const int pos = n + __popcll(b1 & below) + __popcll(b2 & below);
                    if (ne >= 1) ent[pos] = (unsigned short)e0;
                    if (ne == 2) ent[pos + 1] = (unsigned short)e1;
                    n += __popcll(b1) + __popcll(b2);
                }
                const bool ar = __any(any_raw);
                if (lane == 0) {
                    sh_nent = n;
                    sh_raw = ar;
                }
            }
            __syncthreads();
            const int nent = uniform_i(sh_nent);
            const bool has_raw = uniform_i(sh_raw) != 0;

            for (int eb = 0; eb < nent; eb += BE) {
                const int ne = min(BE, nent - eb);
                // ---- node photons: four lanes an entry, each a quarter of the
                // column's samples in order
                if (wv == 0 && has_raw) {
                    // node offsets (entries that are not raw hold M nodes)
                    int cnt = 0;
                    if (lane < ne) {
                        const unsigned en = ent[eb + lane];
                        const int c = en & 127;
                        cnt = (en & kEntRaw) ? kst[c + 1] - kst[c] : M;
                    }
                    int x = cnt;
#pragma unroll
                    for (int o = 1; o < 64; o <<= 1) {
                        const int y = __shfl_up(x, o);
                        if (lane >= o) x += y;
                    }
                    if (lane < ne) noff[lane] = x - cnt;
                    if (lane == ne - 1) noff[ne] = x;
                }
                {
                    const int e = tid >> 2, part = tid & 3;
                    unsigned en = kEntRaw;
                    if (e < ne) en = ent[eb + e];
                    const bool fit = !(en & kEntRaw);
                    const int c = en & 127;
                    double mu[M];
#pragma unroll
                    for (int p = 0; p < M; ++p) mu[p] = 0.0;
                    if (fit) {
                        // Samples in pairs (ks + j, ke - 1 - j), whose tau are
                        // opposite: T_p is even or odd, so a pair costs one
                        // recurrence on its sum and one on its difference, in
                        // steps of T_2.  Groups of four pairs go round the quad's
                        // lanes, so a quad reads 64 consecutive bytes a side.
                        const int ks = kst[c], ke = kst[c + 1];
                        const int J = ke - ks, hJ = J >> 1;
                        const double step = 2.0 * recip((double)(J - 1));
                        const bool test = (en & kEntTest) != 0;
                        const double ar = (double)((int)((en >> 7) & 63) - kMaxH + Y0);
                        auto keep = [&](int k) {  // this sample has the entry's row anchor
                            return !test || floor(horner<DY>(cyr, fma((double)k, dt, t0)) + 0.5) == ar;
                        };
                        auto pair = [&](int j, double pf, double pb) {
                            if (test) {
                                pf = keep(ks + j) ? pf : 0.0;
                                pb = keep(ke - 1 - j) ? pb : 0.0;
                            }
                            const double tau = fma((double)j, step, -1.0);
                            const double w2 = fma(tau + tau, tau, -1.0), w = w2 + w2;  // T_2, 2 T_2
                            double ea = pf + pb, eb = w2 * ea;      // T_0, T_2
                            const double d = pf - pb;
                            double oa = tau * d, ob = fma(w, oa, -oa);  // T_1, T_3
                            mu[0] += ea;
                            mu[1] += oa;
                            mu[2] += eb;
                            mu[3] += ob;
#pragma unroll
                            for (int p = 4; p < M; p += 2) {
                                const double ec = fma(w, eb, -ea), oc = fma(w, ob, -oa);
                                mu[p] += ec;
                                mu[p + 1] += oc;
                                ea = eb;
                                eb = ec;
                                oa = ob;
                                ob = oc;
                            }
                        };
                        // (where registers allow, the next four pairs are loaded
                        // while these are added)
                        constexpr bool kAhead = sizeof(ST) == 4 && DX <= 4;
                        int j = 4 * part;
                        ST vf[4], vb[4];
                        auto fetch = [&](int jj, ST *f, ST *b) {
                            Vec4<ST>::load(spec, ks + jj, f);
                            Vec4<ST>::load(spec, ke - 4 - jj, b);
                        };
                        if (kAhead && j + 4 <= hJ) fetch(j, vf, vb);
                        for (; j + 4 <= hJ; j += 16) {
                            ST nf[4], nb[4];
                            if constexpr (kAhead) fetch(j + 20 <= hJ ? j + 16 : j, nf, nb);
                            else fetch(j, vf, vb);
#pragma unroll
                            for (int e = 0; e < 4; ++e) pair(j + e, (double)vf[e], (double)vb[3 - e]);
                            if constexpr (kAhead) {
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    vf[e] = nf[e];
                                    vb[e] = nb[e];
                                }
                            }
                        }
                        for (; j < hJ; ++j) pair(j, (double)spec[ks + j], (double)spec[ke - 1 - j]);
                        if ((J & 1) && part == 0 && keep(ks + hJ)) {  // the middle one: tau = 0
                            const double phi = (double)spec[ks + hJ];
#pragma unroll
                            for (int p = 0; p < M; p += 2) mu[p] += p & 2 ? -phi : phi;
                        }
                    }
#pragma unroll
                    for (int p = 0; p < M; ++p) mu[p] = quad_sum(mu[p]);
                    // a column with an infinite sample: all its nodes are infinite,
                    // as its samples are one by one
                    if (fit && __builtin_expect(!isfinite(mu[0]), 0)) {
#pragma unroll
                        for (int p = 1; p < M; ++p) mu[p] = 0.0;
                    }
                    if (fit) {
#pragma unroll
                        for (int j = 0; j < (M + 3) / 4; ++j) {
                            const int m = part + 4 * j;
                            if (m >= M) break;
                            // Clenshaw sum of mu_0 / 2 + sum_p mu_p T_p, times 2 / M
                            const double xx = snode[m];
                            double b1 = 0.0, b2 = 0.0;
#pragma unroll
                            for (int p = M - 1; p >= 1; --p) {
                                const double b0 = fma(2.0 * xx, b1, mu[p] - b2);
                                b2 = b1;
                                b1 = b0;
                            }
                            const double sum = fma(xx, b1, 0.5 * mu[0] - b2);
                            sphi[e][m] = (float)(sum * (2.0 / M) * scale);
                        }
                    }
                }
                __syncthreads();
                const int nn = has_raw ? uniform_i(noff[ne]) : ne * M;

                // this thread's node and axis of a chunk: position from its anchor,
                // sigma, photons (worked out one chunk ahead, beside the products)
                float phi;
                double pos, sgm;
                int anchor;
                auto prep = [&](int id) {
                    phi = 0.0f;
                    pos = 0.0;
                    sgm = 1.0;
                    anchor = 0;
                    if (s >= CH || id >= nn) return;
                    int e, m;
                    if (has_raw) {
                        int lo = 0, hi = ne - 1;  // last entry with noff <= id
                        while (lo < hi) {
                            const int mid = (lo + hi + 1) >> 1;
                            if (noff[mid] <= id) lo = mid; else hi = mid - 1;
                        }
                        e = lo;
                        m = id - noff[e];
                    } else {
                        e = id / M;
                        m = id - e * M;
                    }
                    const unsigned en = ent[eb + e];
                    const int c = en & 127;
                    double x, y, ax, ay;
                    if (en & kEntRaw) {
                        const int k = kst[c] + m;
                        const double t = fma((double)k, dt, t0);
                        x = horner<DX>(cxr, t);
                        y = horner<DY>(cyr, t);
                        ax = floor(x + 0.5);
                        ay = floor(y + 0.5);
                        if (xaxis) phi = (float)(spec_at(spec, k) * scale);
                    } else {
                        const int ks = kst[c], ke = kst[c + 1];
                        const double t = fma(node_sample(ks, ke, snode[m]), dt, t0);
                        ax = (double)(X0 - H + c);
                        x = horner<DX>(cxr, t);
                        y = horner<DY>(cyr, t);
                        ay = (double)((int)((en >> 7) & 63) - kMaxH + Y0);
                        if (xaxis) phi = sphi[e][m];
                    }
                    pos = xaxis ? x - ax : y - ay;
                    anchor = (int)(xaxis ? ax : ay);
                    sgm = sigma_axis(F.sxy, F.gx, F.gy, F.gsx, F.gsy, x, y, xaxis ? 0 : 1);
                };
                prep(s);
                for (int c0 = 0; c0 < nn; c0 += CH) {
                    // ---- staging: this thread's node and axis
                    {
                        int nlo = 1, nhi = 0;
                        const bool have = s < CH && c0 + s < nn;
                        if (have) {
                            if (xaxis)
                                stage_axis<TX>(pos, sgm, H, (double)phi, anchor - H - X0, s, buf,
                                               &nlo, &nhi);
                            else
                                stage_axis<TY>(pos, sgm, H, 1.0, anchor - H - Y0, s, ybuf, &nlo,
                                               &nhi);
                        }
                        if (nlo > nhi) nlo = 1, nhi = 0;
                        clear_lines(zlo, zhi, nlo, nhi, s, xaxis ? buf : ybuf);
                        zlo = nlo;
                        zhi = nhi;
                        // (a node without photons reaches none)
                        group_masks(xaxis && phi == 0.0f ? 0u : block_bits(nlo, nhi), lane, wv, smask);
                    }
                    __syncthreads();
                    if (c0 + CH < nn) prep(c0 + CH + s);
                    // ---- products: wave wv takes column block wv
                    tile_products<false, SPAN>(buf, ybuf, nullptr, smask, wv, l16, lg, acc);
                    __syncthreads();
                }
            }
        }
        // Far from a narrow Gaussian's centre the interpolant can pass below zero, by
        // 1e-20 of the photons (sigma 0.6 px, isolated bright samples): w varies by
        // e^(z / sigma) over a column there, and the products' rounding shows from
        // e^15 on.  So where a pixel is negative (rare) and none of the tile's samples
        // is, it is zero.  (An instance of its own, for the frames whose windows reach
        // that far: in every 12-node frame it took 1.6%.)
        if constexpr (NARROW) {
            bool neg = false;
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int q = 0; q < 4; ++q) neg |= acc[rb][q] < 0.0;
            if (neg) sh_neg = 1;
            __syncthreads();
            if (__builtin_expect(uniform_i(sh_neg) != 0, 0)) {
                bool meant = false;
                for (int li = 0; li < count; ++li) {
                    const int tr = uniform_i((int)tlist[li]);
                    const ST *spec = (const ST *)F.tf[tr].spec;
                    const unsigned k1 = segs[tr].k1;
                    for (unsigned k = (unsigned)segs[tr].k0 + tid; k < k1; k += 256)
                        meant |= spec[k] < (ST)0;
                }
                if (meant) sh_neg = 2;
                __syncthreads();
                if (sh_neg == 1) {
#pragma unroll
                    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[rb][q] = acc[rb][q] < 0.0 ? 0.0 : acc[rb][q];
                }
            }
        }
        put_tile(F, X0, Y0, wv, l16, lg, acc);
        __syncthreads();
    }
}

template <int DX, int DY, typename ST, int M, bool NARROW>
hipError_t launch_m(const FrameDev *frames_dev, int precision, const int2 *work, int n_work,
                    int *counter, int *err, int nb, hipStream_t s)
{
    if (precision == E2E_PREC_F64)
        hipLaunchKernelGGL((k_render_sep_fit<DX, DY, ST, M, 4, NARROW>), dim3(nb), dim3(256), 0, s,
                           frames_dev, work, n_work, counter, err);
    else
        hipLaunchKernelGGL((k_render_sep_fit<DX, DY, ST, M, 16, NARROW>), dim3(nb), dim3(256), 0, s,
                           frames_dev, work, n_work, counter, err);
    return hipGetLastError();
}

template <int DX, int DY, typename ST>
hipError_t launch_st(const FrameDev *frames_dev, const KernelCfg &cfg, const int2 *work, int n_work,
                     int *counter, int *err, int nb, hipStream_t s)
{
    const int prec = cfg.precision;
    if (cfg.nodes == 10)
        return launch_m<DX, DY, ST, 10, false>(frames_dev, prec, work, n_work, counter, err, nb, s);
    if (cfg.nodes == 12)
        return launch_m<DX, DY, ST, 12, false>(frames_dev, prec, work, n_work, counter, err, nb, s);
    return launch_m<DX, DY, ST, 12, true>(frames_dev, prec, work, n_work, counter, err, nb, s);
}

template <int DX, int DY>
hipError_t launch_deg(const FrameDev *frames_dev, const KernelCfg &cfg, const int2 *work,
                      int n_work, int *counter, int *err, int nb, hipStream_t s)
{
    if (cfg.spec_f64)
        return launch_st<DX, DY, double>(frames_dev, cfg, work, n_work, counter, err, nb, s);
    return launch_st<DX, DY, float>(frames_dev, cfg, work, n_work, counter, err, nb, s);
}

}  // namespace

hipError_t launch_sep_fit(const FrameDev *frames_dev, const KernelCfg &cfg, const int2 *work,
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
