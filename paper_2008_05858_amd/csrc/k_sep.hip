// Render path for analytic Gaussian PSFs (Sec. 2.1: Gaussian aberration
// model), circular (GAUSS_ERF) or axis-aligned with (sigma_x, sigma_y)
// interpolated across the field (SEPARABLE).  A pixel's weight is the exact
// integral of the Gaussian over the pixel (Sec. 2.2: SFI integrated over the
// pixel area), i.e. a product of normal-CDF differences per axis, over a
// (2H+1)^2 window around floor(x + 1/2), renormalised by the window sum.
//
// Positions are FP64; the CDF differences are evaluated in FP32 on
// pixel-relative offsets (|offset| <= H + 1), each edge through one erfc on
// the side of the distribution where nothing cancels (library erfcf; the
// FP32 variant uses a fitted FP32 normal tail).  One workgroup owns a 16 x 16
// tile and stages one sample's per-axis weights per thread in LDS, aligned
// to the tile's columns and rows (zero outside each window).  Each thread
// adds the products of one or two pixels of one column in sample order (FP64
// sums of FP32 partials over four consecutive samples, or FP32 sums), so the
// result is deterministic and written once.
//
// A tile's samples are a serial chain of chunks, and a small frame has work in
// fewer tiles than the GPU has CUs (a 512 x 256 frame with one trace of 40
// samples a pixel: ~80 tiles of ~1000 samples, 38 us, half of it erfcf and half
// the sums).  So the samples of a tile are cut into at most kSepUnits units of
// whole blocks of 128, each unit's FP64 sum starting at zero and the units
// added in order: the same bits whether one workgroup does all of them or, in
// frames of few tiles, each is a workgroup of its own (k_sep_unit, then
// k_sep_add).
#include "psf_gauss.h"

namespace e2e {

namespace {

// NP pixels per thread (rows tcy + (16 / NP) j of column tcx), 256 / NP
// threads per tile, as many samples staged together, one per thread.  Large
// frames take NP = 2 (the column's weight read shared by two pixels), small
// ones NP = 1 (twice the waves per tile, half the chunks: lower latency).
// Both add every pixel's products in the same groups of four consecutive
// samples, so they give the same bits.
constexpr int kSepSmallTiles = 16384;
constexpr int kSepBlock = 128;   // samples of a block: every chunk is a multiple

// The traces that reach tile row ty, ascending, into tlist, by the first wave;
// *blocks: their blocks of samples in this tile column.  Complete for every
// thread after the caller's next barrier.
__device__ __forceinline__ void list_traces(const SegDev *segs, int ntr, int ty, int lane,
                                            int *tlist, int *sh_count, int *sh_blocks, int *err)
{
    int cnt = 0, nb = 0;
    for (int base = 0; base < ntr; base += 64) {
        const int tr = base + lane;
        bool ok = false;
        int own = 0;
        if (tr < ntr) {
            const SegDev s = segs[tr];
            ok = s.k0 < s.k1 && s.ty0 <= ty && ty <= s.ty1;
            own = (s.k1 - s.k0 + kSepBlock - 1) / kSepBlock;
        }
        const unsigned long long m = __ballot(ok);
        const int pos = cnt + __popcll(m & ((1ull << lane) - 1ull));
        if (ok) {
            if (pos < kMaxTileTraces) {
                tlist[pos] = tr;
                nb += own;
            } else {
                atomicOr(err, kErrTileTraces);
            }
        }
        cnt += __popcll(m);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) nb += __shfl_xor(nb, o);
    if (lane == 0) {
        *sh_count = min(cnt, kMaxTileTraces);
        *sh_blocks = nb;
    }
}

template <int DX, int DY, typename ST, bool SEP, bool ACC64, int NP>
__global__ __launch_bounds__(256 / NP) void k_render_sep(const FrameDev *__restrict__ frames,
                                                         const int2 *__restrict__ work,
                                                         int n_work, int *__restrict__ counter,
                                                         int *__restrict__ err)
{
    constexpr int TS = kSepTile;
    static_assert(TS == 16, "tile-aligned weights are 16 wide");
    static_assert(NP == 1 || NP == 2, "one or two pixels per thread");
    constexpr int kChunk = 256 / NP;
    // per staged sample, its weights on the tile's 16 columns / 16 rows
    // (zero outside its window), stored column-major ([pixel][sample]) so a
    // thread reads four consecutive samples' weights in one 16-byte load
    // (rows padded by 4 floats: the 16 rows read together start on
    // different banks)
    constexpr int RS = kChunk + 4;
    __shared__ __align__(16) float swx[TS][RS];
    __shared__ __align__(16) float swy[TS][RS];
    __shared__ int tlist[kMaxTileTraces];
    __shared__ int sh_count, sh_blocks, sh_item;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    for (int iter = 0;; ++iter) {
        int fi, tile_id;
        if (work == nullptr) {
            if (iter > 0) break;
            fi = 0;
            tile_id = xcd_remap(blockIdx.x, gridDim.x);
        } else {
            if (tid == 0) sh_item = atomicAdd(counter, 1);
            __syncthreads();
            int w = uniform_i(sh_item);
            if (w >= n_work) break;
            int2 wk = work[w];
            fi = uniform_i(wk.x);
            tile_id = uniform_i(wk.y);
        }
        const FrameDev &F = frames[fi];
        const int ntr = F.ntr, H = F.H;
        const int tx = tile_id % F.ntx, ty = tile_id / F.ntx;
        const int X0 = tx * TS, Y0 = ty * TS;
        const SegDev *segs = F.segs + (size_t)tx * ntr;
        if (tid < 64) list_traces(segs, ntr, ty, lane, tlist, &sh_count, &sh_blocks, err);
        __syncthreads();
        const int count = uniform_i(sh_count);
        // blocks of a unit, and the blocks left of the unit at hand
        const int ublk = (uniform_i(sh_blocks) + kSepUnits - 1) / kSepUnits;
        int left = ublk;
        const int tcx = tid % TS, tcy = tid / TS;
        const int pi = X0 + tcx, pj = Y0 + tcy;
        double acc64[NP], unit[NP];
        float acc32[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            acc64[j] = unit[j] = 0.0;
            acc32[j] = 0.0f;
        }

        for (int li = 0; li < count; ++li) {
            const int tr = uniform_i(tlist[li]);
            const TraceDev &T = F.tr[tr];
            const SegDev sg = segs[tr];
            double cxr[DX + 1], cyr[DY + 1];
#pragma unroll
            for (int j = 0; j <= DX; ++j) cxr[j] = T.cx[j];
#pragma unroll
            for (int j = 0; j <= DY; ++j) cyr[j] = T.cy[j];
            double t0, dt;
            trace_affine(T, F.beta, &t0, &dt);
            const float scale = (float)(T.thr * F.flux_scale);
            const ST *spec = (const ST *)F.spec[T.slot];
            for (int kc = sg.k0; kc < sg.k1; kc += kChunk) {
                const int nk = min(kChunk, sg.k1 - kc);
                if (tid < nk) {
                    const int k = kc + tid;
                    double t = fma((double)k, dt, t0);
                    double x = horner<DX>(cxr, t);
                    double y = horner<DY>(cyr, t);
                    double axd = floor(x + 0.5), ayd = floor(y + 0.5);
                    float sgx, sgy;
                    if (SEP) {
                        sigma_at(F.sxy, F.gx, F.gy, F.gsx, F.gsy, x, y, &sgx, &sgy);
                    } else {
                        sgx = sgy = (float)F.sigma;
                    }
                    float phi = (float)spec_at(spec, k) * scale;
                    // the FP32 variant takes the FP32 fitted normal tail
                    axis_weights_tile<TS, RS, !ACC64>((float)(x - axd), sgx, H, phi,
                                                      (int)axd - H - X0, &swx[0][tid]);
                    axis_weights_tile<TS, RS, !ACC64>((float)(y - ayd), sgy, H, 1.0f,
                                                      (int)ayd - H - Y0, &swy[0][tid]);
                } else {
#pragma unroll
                    for (int c = 0; c < TS; ++c) {
                        swx[c][tid] = 0.0f;
                        swy[c][tid] = 0.0f;
                    }
                }
                __syncthreads();
                // every staged sample in order (four per 16-byte read); outside
                // its window both weights' product is 0 and leaves the sum
                // unchanged
                const float4 *px = reinterpret_cast<const float4 *>(swx[tcx]);
                const int nq = (nk + 3) / 4;
                for (int q0 = 0; q0 < nq; q0 += kSepBlock / 4) {  // a block
                    if (ACC64) {
                        if (left == 0) {
#pragma unroll
                            for (int j = 0; j < NP; ++j) {
                                acc64[j] += unit[j];
                                unit[j] = 0.0;
                            }
                            left = ublk;
                        }
                        --left;
                    }
                    const int q1 = min(q0 + kSepBlock / 4, nq);
                    for (int q = q0; q < q1; ++q) {
                        const float4 a = px[q];
#pragma unroll
                        for (int j = 0; j < NP; ++j) {
                            const float4 b =
                                reinterpret_cast<const float4 *>(swy[tcy + (TS / NP) * j])[q];
                            const float v0 = a.x * b.x, v1 = a.y * b.y, v2 = a.z * b.z,
                                        v3 = a.w * b.w;
                            if (ACC64) {
                                // four non-negative products summed in FP32 (relative
                                // error <= 3 ulp of the partial), the partials in FP64
                                unit[j] += (double)(((v0 + v1) + v2) + v3);
                            } else {
                                acc32[j] += v0;
                                acc32[j] += v1;
                                acc32[j] += v2;
                                acc32[j] += v3;
                            }
                        }
                    }
                }
                __syncthreads();
            }
        }
        if (pi < F.nx) {
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int row = pj + (TS / NP) * j;
                if (row >= F.ny) continue;
                double v = ACC64 ? acc64[j] + unit[j] : (double)acc32[j];
                size_t o = (size_t)row * F.nx + pi;
                if (F.out_f64) ((double *)F.out)[o] = v;
                else ((float *)F.out)[o] = (float)v;
            }
        }
        __syncthreads();
    }
}

// One unit of one tile: thread s < 128 stages sample s of a block on the
// tile's columns, thread 128 + s on its rows; then each thread sums its pixel
// over the block.  The unit's sum goes to part[item][unit][pixel].
template <int DX, int DY, typename ST, bool SEP>
__global__ __launch_bounds__(256) void k_sep_unit(const FrameDev *__restrict__ frames,
                                                  const int2 *__restrict__ work, SepParts parts,
                                                  int *__restrict__ err)
{
    constexpr int TS = kSepTile;
    constexpr int RS = kSepBlock + 4;
    __shared__ __align__(16) float swx[TS][RS];
    __shared__ __align__(16) float swy[TS][RS];
    __shared__ int tlist[kMaxTileTraces];
    __shared__ int sh_count, sh_blocks;

    const int tid = threadIdx.x;
    const int item = blockIdx.x / kSepUnits, u = blockIdx.x % kSepUnits;
    const int fi = work ? uniform_i(work[item].x) : 0;
    const int tile_id = work ? uniform_i(work[item].y) : item;
    const FrameDev &F = frames[fi];
    const int ntr = F.ntr, H = F.H;
    const int tx = tile_id % F.ntx, ty = tile_id / F.ntx;
    const int X0 = tx * TS, Y0 = ty * TS;
    const SegDev *segs = F.segs + (size_t)tx * ntr;
    if (tid < 64) list_traces(segs, ntr, ty, tid, tlist, &sh_count, &sh_blocks, err);
    __syncthreads();
    const int count = uniform_i(sh_count), blocks = uniform_i(sh_blocks);
    const int ublk = (blocks + kSepUnits - 1) / kSepUnits;
    if (u == 0 && tid == 0) parts.units[item] = ublk == 0 ? 0 : (blocks + ublk - 1) / ublk;
    const int b0 = u * ublk, b1 = min(b0 + ublk, blocks);
    if (b0 >= b1) return;
    const int tcx = tid % TS, tcy = tid / TS;
    const int s = tid % kSepBlock;
    const bool xaxis = tid < kSepBlock;
    double unit = 0.0;
    int b = 0;  // first block of the trace
    for (int li = 0; li < count && b < b1; ++li) {
        const int tr = uniform_i(tlist[li]);
        const SegDev sg = segs[tr];
        const int nb = (sg.k1 - sg.k0 + kSepBlock - 1) / kSepBlock;
        const int f0 = max(b0 - b, 0), f1 = min(b1 - b, nb);
        b += nb;
        if (f0 >= f1) continue;
        const TraceDev &T = F.tr[tr];
        double t0, dt;
        trace_affine(T, F.beta, &t0, &dt);
        const float scale = (float)(T.thr * F.flux_scale);
        const ST *spec = (const ST *)F.spec[T.slot];
        for (int f = f0; f < f1; ++f) {
            const int kc = sg.k0 + f * kSepBlock;
            const int nk = min(kSepBlock, sg.k1 - kc);
            float *const w = xaxis ? &swx[0][s] : &swy[0][s];
            if (s < nk) {
                const int k = kc + s;
                double cxr[DX + 1], cyr[DY + 1];
#pragma unroll
                for (int j = 0; j <= DX; ++j) cxr[j] = T.cx[j];
#pragma unroll
                for (int j = 0; j <= DY; ++j) cyr[j] = T.cy[j];
                const double t = fma((double)k, dt, t0);
                const double x = horner<DX>(cxr, t), y = horner<DY>(cyr, t);
                float sgx, sgy;
                if (SEP) sigma_at(F.sxy, F.gx, F.gy, F.gsx, F.gsy, x, y, &sgx, &sgy);
                else sgx = sgy = (float)F.sigma;
                const double p = xaxis ? x : y, a = floor(p + 0.5);
                const float phi = xaxis ? (float)spec_at(spec, k) * scale : 1.0f;
                axis_weights_tile<TS, RS, false>((float)(p - a), xaxis ? sgx : sgy, H, phi,
                                                 (int)a - H - (xaxis ? X0 : Y0), w);
            } else {
#pragma unroll
                for (int c = 0; c < TS; ++c) w[c * RS] = 0.0f;
            }
            __syncthreads();
            const float4 *px = reinterpret_cast<const float4 *>(swx[tcx]);
            const float4 *py = reinterpret_cast<const float4 *>(swy[tcy]);
            for (int q = 0; q < (nk + 3) / 4; ++q) {
                const float4 a = px[q], w4 = py[q];
                const float v0 = a.x * w4.x, v1 = a.y * w4.y, v2 = a.z * w4.z, v3 = a.w * w4.w;
                unit += (double)(((v0 + v1) + v2) + v3);
            }
            __syncthreads();
        }
    }
    parts.part[((size_t)item * kSepUnits + u) * 256 + tid] = unit;
}

// Every pixel's units, added in order, and the frame written.
__global__ __launch_bounds__(256) void k_sep_add(const FrameDev *__restrict__ frames,
                                                 const int2 *__restrict__ work, SepParts parts)
{
    constexpr int TS = kSepTile;
    const int item = blockIdx.x, tid = threadIdx.x;
    const int fi = work ? uniform_i(work[item].x) : 0;
    const int tile_id = work ? uniform_i(work[item].y) : item;
    const int n = uniform_i(parts.units[item]);
    const double *p = parts.part + (size_t)item * kSepUnits * 256 + tid;
    double v[kSepUnits], acc = 0.0;
#pragma unroll
    for (int u = 0; u < kSepUnits; ++u) v[u] = u < n ? p[u * 256] : 0.0;
#pragma unroll
    for (int u = 0; u < kSepUnits; ++u)
        if (u < n) acc += v[u];
    const FrameDev &F = frames[fi];
    const int gx = (tile_id % F.ntx) * TS + tid % TS, gy = (tile_id / F.ntx) * TS + tid / TS;
    if (gx >= F.nx || gy >= F.ny) return;
    const size_t o = (size_t)gy * F.nx + gx;
    if (F.out_f64) ((double *)F.out)[o] = acc;
    else ((float *)F.out)[o] = (float)acc;
}

template <int DX, int DY, typename ST>
hipError_t launch_units(const FrameDev *frames_dev, const KernelCfg &cfg, bool sep,
                        const int2 *work, int n_items, int *err, hipStream_t s)
{
    const dim3 grid((unsigned)n_items * kSepUnits);
    if (sep)
        hipLaunchKernelGGL((k_sep_unit<DX, DY, ST, true>), grid, dim3(256), 0, s, frames_dev, work,
                           cfg.parts, err);
    else
        hipLaunchKernelGGL((k_sep_unit<DX, DY, ST, false>), grid, dim3(256), 0, s, frames_dev, work,
                           cfg.parts, err);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sep_add, dim3(n_items), dim3(256), 0, s, frames_dev, work, cfg.parts);
    return hipGetLastError();
}

template <int DX, int DY, typename ST, int NP>
hipError_t launch_np(const FrameDev *frames_dev, bool acc64, bool sep, const int2 *work,
                     int n_work, int *counter, int *err, hipStream_t s)
{
    // plain: one workgroup per tile; persistent: 4096 waves, 16 per CU
    constexpr int NT = 256 / NP;
    const int cap = 2048 * 256 / (NT * 2);
    const int nb = work == nullptr ? n_work : (n_work < cap ? n_work : cap);
    if (sep) {
        if (acc64)
            hipLaunchKernelGGL((k_render_sep<DX, DY, ST, true, true, NP>), dim3(nb), dim3(NT), 0,
                               s, frames_dev, work, n_work, counter, err);
        else
            hipLaunchKernelGGL((k_render_sep<DX, DY, ST, true, false, NP>), dim3(nb), dim3(NT),
                               0, s, frames_dev, work, n_work, counter, err);
    } else {
        if (acc64)
            hipLaunchKernelGGL((k_render_sep<DX, DY, ST, false, true, NP>), dim3(nb), dim3(NT),
                               0, s, frames_dev, work, n_work, counter, err);
        else
            hipLaunchKernelGGL((k_render_sep<DX, DY, ST, false, false, NP>), dim3(nb), dim3(NT),
                               0, s, frames_dev, work, n_work, counter, err);
    }
    return hipGetLastError();
}

template <int DX, int DY, typename ST>
hipError_t launch_st(const FrameDev *frames_dev, const KernelCfg &cfg, bool sep,
                     const int2 *work, int n_items, int *counter, int *err, hipStream_t s)
{
    const bool acc64 = cfg.precision != E2E_PREC_F32;
    if (acc64 && cfg.parts.part)
        return launch_units<DX, DY, ST>(frames_dev, cfg, sep, work, n_items, err, s);
    if (n_items < kSepSmallTiles)
        return launch_np<DX, DY, ST, 1>(frames_dev, acc64, sep, work, n_items, counter, err, s);
    return launch_np<DX, DY, ST, 2>(frames_dev, acc64, sep, work, n_items, counter, err, s);
}

template <int DX, int DY>
hipError_t launch_deg(const FrameDev *frames_dev, const KernelCfg &cfg, bool sep,
                      const int2 *work, int n_items, int *counter, int *err, hipStream_t s)
{
    if (cfg.spec_f64)
        return launch_st<DX, DY, double>(frames_dev, cfg, sep, work, n_items, counter, err, s);
    return launch_st<DX, DY, float>(frames_dev, cfg, sep, work, n_items, counter, err, s);
}

}  // namespace

// sep is read from the first frame's PSF kind on the host side and passed
// through cfg.kw: 1 = SEPARABLE, 0 = GAUSS_ERF.
hipError_t launch_sep(const FrameDev *frames_dev, const KernelCfg &cfg, const int2 *work,
                      int n_work, int *counter, int *err, hipStream_t s)
{
    // tiles of the plain launch, or work items of the persistent one
    const int n_items = work == nullptr ? cfg.plain_tiles : n_work;
    if (n_items <= 0) return hipSuccess;
    bool sep = cfg.kw != 0;
    if (cfg.degx <= 3 && cfg.degy <= 2)
        return launch_deg<3, 2>(frames_dev, cfg, sep, work, n_items, counter, err, s);
    if (cfg.degx <= 4 && cfg.degy <= 3)
        return launch_deg<4, 3>(frames_dev, cfg, sep, work, n_items, counter, err, s);
    return launch_deg<7, 7>(frames_dev, cfg, sep, work, n_items, counter, err, s);
}

}  // namespace e2e
