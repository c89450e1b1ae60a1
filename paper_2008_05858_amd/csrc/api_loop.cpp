// C ABI of the closing-the-loop steps (Sec. 1, Sec. 4.2): e2e_extract and
// e2e_ccf.  Argument checks, staging of host buffers, the template
// smoothing widths, launches, and the parabola vertex of the summed CCF.
#include <cmath>
#include <cstring>
#include <map>
#include <tuple>
#include <vector>

#include "api_internal.h"

namespace e2e {
hipError_t launch_extract(const TraceDev *trs, int ntr, int nx, int ny, const void *frame,
                          int f64, double A, double *flux, double *edges, hipStream_t s);
hipError_t launch_smooth3(const void *lt_dev, int n_tmpl, int64_t nmax, int wmax, int f64,
                          hipStream_t s);
int loop_max_width();
bool loop_needs_p(int w);
int loop_max_templates();
hipError_t launch_ccf_mean(const TraceDev *trs, const void *tl_dev, int n_tr, const void *lt_dev,
                           int nx, const double *flux, const double *flat, const double *edges,
                           double v0, double dv, int nv, double *mean, hipStream_t s);
hipError_t launch_ccf(const TraceDev *trs, const void *tl_dev, int n_tr, int ntr, const void *lt_dev,
                      int nx, double spp, double vspan, const double *flux, const double *flat,
                      const double *edges, double v0, double dv, int nv, const double *mean,
                      double *part, double *C, hipStream_t s);
hipError_t launch_ccf_total(const double *part, int ntr, int nx, int nv, double *C, double *tot,
                            hipStream_t s);
size_t ccf_part_bytes(int nx, int ntr, int nv);
size_t loop_template_bytes();
size_t loop_trace_bytes();
void loop_template_fill(void *dst, const void *tmpl, double *P, double *X, int64_t n, int w);
void loop_trace_fill(void *dst, int trace, int tmpl);
}  // namespace e2e

using namespace e2e;

namespace {

// Device buffers of one call, released on every exit path.
struct Bufs {
    e2e_ctx *ctx;
    std::vector<void *> p;
    explicit Bufs(e2e_ctx *c) : ctx(c) {}
    ~Bufs()
    {
        for (void *q : p) hipFree(q);
    }
    hipError_t get(void **out, size_t bytes)
    {
        hipError_t e = dev_malloc(ctx, out, bytes > 0 ? bytes : 16, false);
        if (e == hipSuccess) p.push_back(*out);
        return e;
    }
};

// The workspace of a CCF, kept by the context between calls where its budget has
// the room: one buffer of at most kLoopKeep bytes, taken by a call and put back when
// its stream has passed its kernels (a call that finds none, as beside another one,
// allocates its own).  Allocating 200 MB and freeing it (which waits for the whole
// device) took 0.4 ms of a 3.0 ms call.
constexpr size_t kLoopKeep = (size_t)256 << 20;
struct KeptBuf {
    e2e_ctx *ctx;
    void *p = nullptr;
    size_t cap = 0;
    explicit KeptBuf(e2e_ctx *c) : ctx(c) {}
    KeptBuf(const KeptBuf &) = delete;
    hipError_t get(size_t need)
    {
        {
            std::lock_guard<std::mutex> lk(ctx->mu);
            std::swap(p, ctx->loop_ws);
            std::swap(cap, ctx->loop_cap);
            ctx->kept -= cap;
        }
        if (p && cap >= need) return hipSuccess;
        if (p) hipFree(p);
        p = nullptr;
        cap = need;
        return dev_malloc(ctx, &p, need, false);
    }
    ~KeptBuf()
    {
        if (!p) return;
        if (cap <= kLoopKeep) {
            std::lock_guard<std::mutex> lk(ctx->mu);
            if (!ctx->loop_ws && fits_beside(ctx, cap)) {
                ctx->kept += cap;
                std::swap(p, ctx->loop_ws);
                std::swap(cap, ctx->loop_cap);
            }
        }
        if (p) hipFree(p);
    }
};

// Holds a reference on a format for the duration of a call, so that
// e2e_format_free reports E2E_EBUSY instead of freeing it underneath.
struct FormatRef {
    e2e_ctx *ctx;
    FormatRes *F = nullptr;
    FormatRef(e2e_ctx *c, e2e_format_id id) : ctx(c)
    {
        std::lock_guard<std::mutex> lk(ctx->mu);
        auto it = ctx->fmts.find(id);
        if (it == ctx->fmts.end()) return;
        F = it->second;
        F->refs++;
    }
    ~FormatRef()
    {
        if (!F) return;
        std::lock_guard<std::mutex> lk(ctx->mu);
        F->refs--;
    }
};

double horner_host(const double *c, int deg, double t)
{
    double v = c[deg];
    for (int j = deg - 1; j >= 0; --j) v = v * t + c[j];
    return v;
}

}  // namespace

extern "C" e2e_status e2e_extract(e2e_ctx *ctx, e2e_format_id fmt, const void *frame,
                                  int32_t dtype, double A, double *flux, double *edges,
                                  int32_t on_device, void *stream)
{
    if (!ctx || !frame || !flux || !edges) return fail(E2E_EINVAL, "e2e_extract: NULL argument");
    if (dtype != E2E_F32 && dtype != E2E_F64) return fail(E2E_EINVAL, "dtype=%d", dtype);
    if (!(std::isfinite(A) && A > 0.0 && A <= 1e6))
        return fail(E2E_EINVAL, "aperture_half_px=%g", A);
    FormatRef ref(ctx, fmt);
    FormatRes *F = ref.F;
    if (!F) return fail(E2E_ENOTFOUND, "format %llu not found", (unsigned long long)fmt);
    hipSetDevice(ctx->dev);
    hipStream_t s = stream ? (hipStream_t)stream : ctx->stream;
    const size_t npx = (size_t)F->nx * F->ny, fb = npx * (dtype == E2E_F64 ? 8 : 4);
    const size_t eb = (size_t)F->ntr * F->nx * 8, lb = (size_t)F->ntr * (F->nx + 1) * 8;
    Bufs B(ctx);
    const void *fd = frame;
    double *ed = flux, *ld = edges;
    hipError_t e = hipSuccess;
    if (!on_device) {
        void *a, *b, *c;
        if ((e = B.get(&a, fb)) != hipSuccess || (e = B.get(&b, eb)) != hipSuccess ||
            (e = B.get(&c, lb)) != hipSuccess)
            return hip_fail(e, "extraction buffers");
        if ((e = hipMemcpyAsync(a, frame, fb, hipMemcpyHostToDevice, s)) != hipSuccess)
            return hip_fail(e, "frame upload");
        fd = a;
        ed = (double *)b;
        ld = (double *)c;
    }
    prof_begin(ctx, s, "extract");
    e = launch_extract(F->dev, F->ntr, F->nx, F->ny, fd, dtype == E2E_F64, A, ed, ld, s);
    prof_end(ctx, s);
    if (e == hipSuccess && !on_device) {
        e = hipMemcpyAsync(flux, ed, eb, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipMemcpyAsync(edges, ld, lb, hipMemcpyDeviceToHost, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "e2e_extract");
    return E2E_OK;
}

extern "C" e2e_status e2e_ccf(e2e_ctx *ctx, e2e_format_id fmt, const e2e_ccf_req *r,
                              double *rv_out)
{
    if (!ctx || !r || !rv_out || !r->flux || !r->edges || !r->templates)
        return fail(E2E_EINVAL, "e2e_ccf: NULL argument");
    if (r->template_dtype != E2E_F32 && r->template_dtype != E2E_F64)
        return fail(E2E_EINVAL, "template_dtype=%d", r->template_dtype);
    if (r->n_v < 3) return fail(E2E_EINVAL, "n_v=%d (needs >= 3)", r->n_v);
    if (!(std::isfinite(r->dv_mps) && r->dv_mps != 0.0) || !std::isfinite(r->v0_mps))
        return fail(E2E_EINVAL, "e2e_ccf: velocity grid");
    const double vmax = std::fmax(std::fabs(r->v0_mps), std::fabs(r->v0_mps + (r->n_v - 1) * r->dv_mps));
    if (vmax > 1.5e7) return fail(E2E_EINVAL, "e2e_ccf: |v| above 1.5e7 m/s");
    if (!(std::isfinite(r->smooth_px) && r->smooth_px > 0.0))
        return fail(E2E_EINVAL, "smooth_px=%g", r->smooth_px);
    FormatRef ref(ctx, fmt);
    FormatRes *F = ref.F;
    if (!F) return fail(E2E_ENOTFOUND, "format %llu not found", (unsigned long long)fmt);
    if (r->n_templates < F->nslots)
        return fail(E2E_EINVAL, "n_templates=%d, the format uses %d", r->n_templates, F->nslots);
    hipSetDevice(ctx->dev);
    hipStream_t s = r->hip_stream ? (hipStream_t)r->hip_stream : ctx->stream;
    const int ntr = F->ntr, nx = F->nx, nv = r->n_v;
    const size_t esz = r->template_dtype == E2E_F64 ? 8 : 4;
    const size_t eb = (size_t)ntr * nx * 8, lb = (size_t)ntr * (nx + 1) * 8;
    Bufs B(ctx);
    hipError_t e = hipSuccess;
    const double *fd = r->flux, *fl = r->flat, *ld = r->edges;
    std::vector<const void *> tmpl(F->nslots, nullptr);
    for (auto &T : F->host) {
        if (!r->templates[T.slot]) return fail(E2E_EINVAL, "template of slot %d is NULL", T.slot);
        tmpl[T.slot] = r->templates[T.slot];
    }
    if (!r->on_device) {
        void *a, *b, *c = nullptr;
        if ((e = B.get(&a, eb)) != hipSuccess || (e = B.get(&b, lb)) != hipSuccess ||
            (r->flat && (e = B.get(&c, eb)) != hipSuccess))
            return hip_fail(e, "ccf buffers");
        if ((e = hipMemcpyAsync(a, r->flux, eb, hipMemcpyHostToDevice, s)) != hipSuccess ||
            (e = hipMemcpyAsync(b, r->edges, lb, hipMemcpyHostToDevice, s)) != hipSuccess ||
            (r->flat && (e = hipMemcpyAsync(c, r->flat, eb, hipMemcpyHostToDevice, s)) !=
                            hipSuccess))
            return hip_fail(e, "ccf upload");
        fd = (const double *)a;
        ld = (const double *)b;
        fl = (const double *)c;
        std::vector<int64_t> len(F->nslots, 0);
        for (auto &T : F->host) len[T.slot] = std::max<int64_t>(len[T.slot], T.n);
        for (int q = 0; q < F->nslots; ++q) {
            if (!tmpl[q]) continue;
            void *d;
            if ((e = B.get(&d, (size_t)len[q] * esz)) != hipSuccess) return hip_fail(e, "template");
            if ((e = hipMemcpyAsync(d, tmpl[q], (size_t)len[q] * esz, hipMemcpyHostToDevice,
                                    s)) != hipSuccess)
                return hip_fail(e, "template upload");
            tmpl[q] = d;
        }
    }
    // moving-mean width of each trace: the odd integer nearest sqrt(4 s^2 + 1),
    // s = smooth_px samples-per-pixel
    std::vector<int> w(ntr);
    std::vector<double> spans(ntr);
    int64_t nmax = 0;
    for (int t = 0; t < ntr; ++t) {
        const TraceDev &T = F->host[t];
        const double span = horner_host(T.cx, kNCoef - 1, 1.0) - horner_host(T.cx, kNCoef - 1, -1.0);
        spans[t] = span;
        const double sg = r->smooth_px * (double)T.n / span;
        int wi = (int)std::floor(std::sqrt(4.0 * sg * sg + 1.0) + 0.5);
        if (wi % 2 == 0) wi += 1;
        w[t] = std::max(1, wi);
        if (w[t] > loop_max_width())
            return fail(E2E_EINVAL, "e2e_ccf: smoothing window of trace %d is %d samples (max %d)",
                        t, w[t], loop_max_width());
        nmax = std::max<int64_t>(nmax, T.n);
    }
    // templates to smooth: one for each (spectrum slot, length, width) in use;
    // the slices of a fiber share theirs.  tmpl_of[t]: that of trace t.
    struct Tmpl {
        int slot, w;
        int64_t n;
        std::vector<int> traces;
    };
    std::vector<Tmpl> uniq;
    std::map<std::tuple<int, int, int64_t>, int> seen;
    for (int t = 0; t < ntr; ++t) {
        const TraceDev &T = F->host[t];
        auto it = seen.emplace(std::make_tuple(T.slot, w[t], (int64_t)T.n), (int)uniq.size());
        if (it.second) uniq.push_back({T.slot, w[t], T.n, {}});
        uniq[it.first->second].traces.push_back(t);
    }
    // as many at a time as 192 MB of smoothed samples hold (they stay in the
    // memory-side cache between the two kernels), and all the tables in one upload
    bool wide = false;
    for (auto &u : uniq) wide |= loop_needs_p(u.w);
    const size_t half = ((size_t)nmax + 1) & ~(size_t)1;  // even: the CCF loads 16 bytes
    const size_t stride = half * (wide ? 2 : 1);
    const int nu = (int)uniq.size();
    const int G = (int)std::max<size_t>(
        1, std::min<size_t>(std::min(nu, loop_max_templates()), ((size_t)192 << 20) / (stride * 8)));
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const size_t b_tm = up(nu * loop_template_bytes()), b_tl = up(ntr * loop_trace_bytes());
    const size_t b_mean = up((size_t)ntr * 8), b_tot = up((size_t)nv * 8);
    const size_t b_C = up((size_t)ntr * nv * 8), b_part = up(ccf_part_bytes(nx, ntr, nv));
    KeptBuf kept(ctx);
    if ((e = kept.get(b_tm + b_tl + b_mean + b_tot + b_C + b_part + G * stride * 8)) != hipSuccess)
        return hip_fail(e, "ccf workspace");
    char *const ws = (char *)kept.p;
    char *const tm = ws, *const tl = tm + b_tm;
    double *const mean = (double *)(tl + b_tl), *const tot_d = (double *)(tl + b_tl + b_mean);
    double *const Cd = (double *)((char *)tot_d + b_tot), *const part = (double *)((char *)Cd + b_C);
    double *const work = (double *)((char *)part + b_part);
    std::vector<char> table(b_tm + b_tl);
    int at = 0;
    for (int u = 0; u < nu; ++u) {
        double *base = work + (size_t)(u % G) * stride;
        loop_template_fill(table.data() + u * loop_template_bytes(), tmpl[uniq[u].slot], base + half, base,
                           uniq[u].n, uniq[u].w);
        for (int t : uniq[u].traces) loop_trace_fill(table.data() + b_tm + at++ * loop_trace_bytes(), t, u);
    }
    e = hipMemcpyAsync(tm, table.data(), table.size(), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) {
        prof_begin(ctx, s, "ccf");
        e = launch_ccf_mean(F->dev, tl, ntr, tm, nx, fd, fl, ld, r->v0_mps, r->dv_mps, nv, mean, s);
        prof_end(ctx, s);
    }
    double *const Cout = r->ccf_out && r->on_device ? r->ccf_out : Cd;
    at = 0;
    for (int u0 = 0; u0 < nu && e == hipSuccess; u0 += G) {
        const int g = std::min(G, nu - u0);
        int64_t ng = 0;
        int wg = 1, nt = 0;
        double spp = 0.0, vspan = 0.0;  // samples a column, samples the velocities span
        for (int u = u0; u < u0 + g; ++u) {
            ng = std::max(ng, uniq[u].n);
            wg = std::max(wg, uniq[u].w);
            nt += (int)uniq[u].traces.size();
            for (int t : uniq[u].traces) {
                const TraceDev &T = F->host[t];
                spp = std::max(spp, 1.1 * (double)T.n / spans[t]);
                vspan = std::max(vspan, (nv - 1) * std::fabs(r->dv_mps) / 299792458.0 * T.lmax *
                                            (double)T.n / (T.lmax - T.lmin));
            }
        }
        prof_begin(ctx, s, "template_smooth");
        e = launch_smooth3(tm + u0 * loop_template_bytes(), g, ng, wg, r->template_dtype == E2E_F64, s);
        prof_end(ctx, s);
        if (e != hipSuccess) break;
        prof_begin(ctx, s, "ccf");
        e = launch_ccf(F->dev, tl + at * loop_trace_bytes(), nt, ntr, tm, nx, spp, vspan, fd, fl, ld,
                       r->v0_mps, r->dv_mps, nv, mean, part, Cout, s);
        prof_end(ctx, s);
        at += nt;
    }
    // the sums over the columns' runs and over the traces, each in order
    if (e == hipSuccess) e = launch_ccf_total(part, ntr, nx, nv, Cout, tot_d, s);
    std::vector<double> tot(nv);
    if (e == hipSuccess) e = hipMemcpyAsync(tot.data(), tot_d, nv * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess && r->ccf_out && !r->on_device)
        e = hipMemcpyAsync(r->ccf_out, Cd, (size_t)ntr * nv * 8, hipMemcpyDeviceToHost, s);
    // (also before an error return: the upload reads `table` until it is done)
    const hipError_t es = hipStreamSynchronize(s);
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) return hip_fail(e, "e2e_ccf");
    // parabola vertex of the summed CCF
    int kb = 1;
    for (int k = 1; k < nv - 1; ++k)
        if (tot[k] > tot[kb]) kb = k;
    const double ym = tot[kb - 1], y0 = tot[kb], yp = tot[kb + 1];
    const double den = ym - 2.0 * y0 + yp;
    const double off = den != 0.0 ? 0.5 * (ym - yp) / den : 0.0;
    *rv_out = r->v0_mps + r->dv_mps * ((double)kb + off);
    return E2E_OK;
}
