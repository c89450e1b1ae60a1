// Shared by the render kernels that multiply separable terms on the matrix
// cores (k_sep_fit.hip, k_sfi_terms.hip): a 64 x 32 pixel tile, chunks of 120
// nodes whose column rows (x) and row rows (y) are staged in LDS in operand
// layout, F += Gy^T Gx by v_mfma_f32_16x16x4_f32, FP32 partials of 4, 8 or 16
// nodes added to FP64 sums (each kernel says which it takes, and why).
#pragma once

#include "psf_gauss.h"

namespace e2e {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kStageTX = 64, kStageTY = 32;
static_assert(kMfmaTW == kStageTX && kMfmaTH == kStageTY && kSfiTW == kStageTX && kSfiTH == kStageTY,
              "tile geometry of both kernels");
constexpr int CH = 120;                // nodes per chunk
constexpr int LS = CH + 4;             // floats of a line in LDS, see lds_at

// Float index of (pixel line p, node s): the operands of one chunk in LDS are
// [line][node] FP32 weights, four floats of zeros after each line.  Lines are
// 124 floats apart, so the 16 lines that a fragment read touches start on
// different banks and a thread's writes go down the lines at a fixed step.
__device__ __forceinline__ int lds_at(int p, int s) { return p * LS + s; }

// 1 / v for v > 0: the hardware reciprocal and two Newton steps
__device__ __forceinline__ double recip(double v)
{
    double r = __builtin_amdgcn_rcp(v);
    r = fma(r, fma(-v, r, 1.0), r);
    return fma(r, fma(-v, r, 1.0), r);
}

// exp(x) for x in [-0.4, 0]: Taylor to x^9 (truncation below 3e-11)
__device__ __forceinline__ double exp_small(double x)
{
    double p = fma(x, 1.0 / 362880.0, 1.0 / 40320.0);
    p = fma(p, x, 1.0 / 5040.0);
    p = fma(p, x, 1.0 / 720.0);
    p = fma(p, x, 1.0 / 120.0);
    p = fma(p, x, 1.0 / 24.0);
    p = fma(p, x, 1.0 / 6.0);
    p = fma(p, x, 0.5);
    p = fma(p, x, 1.0);
    return fma(p, x, 1.0);
}

// exp(x) for |x| < 700: 2^n times exp of the remainder, |r| <= ln2 / 2
// (Taylor to r^9, relative error below 1e-11)
__device__ __forceinline__ double exp_mid(double x)
{
    const double n = rint(x * 1.4426950408889634);
    const double r = fma(n, -0.6931471805599453, x);
    return ldexp(exp_small(r), (int)n);
}

// zero lines [zlo, zhi] of sample slot s except [nlo, nhi]
__device__ __forceinline__ void clear_lines(int zlo, int zhi, int nlo, int nhi, int s,
                                            float *b)
{
    const bool none = nlo > nhi;
    const int e1 = none ? zhi : min(zhi, nlo - 1);
    for (int p = zlo; p <= e1; ++p) b[lds_at(p, s)] = 0.0f;
    if (!none)
        for (int p = max(zlo, nhi + 1); p <= zhi; ++p) b[lds_at(p, s)] = 0.0f;
}

// 16-line blocks covered by lines [lo, hi]
__device__ __forceinline__ unsigned block_bits(int lo, int hi)
{
    if (lo > hi) return 0u;
    const int b0 = lo >> 4, b1 = hi >> 4;
    return ((2u << b1) - 1u) & ~((1u << b0) - 1u);
}

// The 16-line blocks that each group of 32 nodes of a chunk reaches, by ballots
// over the wave (waves 0-1: x lines, 2-3: y lines; lane = node slot mod 64).
__device__ __forceinline__ void group_masks(unsigned bits, int lane, int wv, unsigned (*smask)[2])
{
    unsigned ma = 0u, mb = 0u;  // nodes 0 .. 31 and 32 .. 63 of the wave
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const unsigned long long w = __ballot((bits >> q) & 1u);
        ma |= (unsigned)w != 0u ? 1u << q : 0u;
        mb |= (unsigned)(w >> 32) != 0u ? 1u << q : 0u;
    }
    if (lane < 2) smask[2 * (wv & 1) + lane][wv >> 1] = lane ? mb : ma;
}

// All lines of both axes to zero (256 threads, 16-byte words).
__device__ __forceinline__ void zero_lines(float *buf, int tid)
{
    static_assert((kStageTX + kStageTY) * LS % 4 == 0, "zeroed by 16-byte words");
    const uint4 zz = {0u, 0u, 0u, 0u};
    uint4 *b4 = reinterpret_cast<uint4 *>(buf);
    for (int q = tid; q < (kStageTX + kStageTY) * LS / 4; q += 256) b4[q] = zz;
}

// Traces whose segments reach tile row ty, ascending, into tlist: 256 tested at
// a time, their counts passed between the waves through smask.  The list is
// complete for every thread after the caller's next barrier.
__device__ __forceinline__ int tile_traces(const SegDev *segs, int ntr, int ty, int tid,
                                           unsigned (*smask)[2], unsigned short *tlist, int *err)
{
    const int lane = tid & 63, wv = tid >> 6;
    int count = 0;
    for (int base = 0; base < ntr; base += 256) {
        const int tr = base + tid;
        bool ok = false;
        if (tr < ntr) {
            const SegDev sv = segs[tr];
            ok = sv.k0 < sv.k1 && sv.ty0 <= ty && ty <= sv.ty1;
        }
        const unsigned long long m = __ballot(ok);
        const int par = (base >> 8) & 1;  // two sets of counts: one barrier a turn
        if (lane == 0) smask[wv][par] = (unsigned)__popcll(m);
        __syncthreads();
        int pos = count + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const int v = (int)smask[w][par];
            pos += w < wv ? v : 0;
            count += v;
        }
        if (ok) {
            if (pos < kMaxTileTraces) tlist[pos] = (unsigned short)tr;
            else atomicOr(err, kErrTileTraces);
        }
    }
    return uniform_i(min(count, kMaxTileTraces));
}

// The products of one staged chunk: wave wv adds column block wv (rows 4 lg + q
// of row block rb, column l16) into acc, SPAN nodes (4, 8 or 16) to an FP32 partial.
// SCALED: each node's x row times scl[node].
template <bool SCALED, int SPAN>
__device__ __forceinline__ void tile_products(const float *buf, const float *ybuf, const float *scl,
                                              const unsigned (*smask)[2], int wv, int l16, int lg,
                                              double (*acc)[4])
{
    const float *const bx = buf + (16 * wv + l16) * LS + 4 * lg;
    const float *const ay = ybuf + l16 * LS + 4 * lg;
    // the chunk's last 8 nodes fill half a group of 16: the lanes of its other
    // half read the zeros behind the line
    const int last = CH - 8 + (lg > 2 ? -4 : 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const unsigned mx = (unsigned)uniform_i((int)smask[j][0]);
        const unsigned my = (unsigned)uniform_i((int)smask[j][1]);
        if (!((mx >> wv) & 1u) || my == 0u) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // 16 nodes: lane group lg holds 4 lg .. + 3
            const int g = j == 3 && h == 1 ? last : 32 * j + 16 * h;
            f4 bv = *reinterpret_cast<const f4 *>(bx + g);
            if constexpr (SCALED) bv *= *reinterpret_cast<const f4 *>(scl + 4 * lg + g);
#pragma unroll
            for (int rb = 0; rb < 2; ++rb) {
                if (!((my >> rb) & 1u)) continue;
                const f4 av = *reinterpret_cast<const f4 *>(ay + 16 * rb * LS + g);
#pragma unroll
                for (int p = 0; p < 16 / SPAN; ++p) {
                    f4 part = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = p * SPAN / 4; q < (p + 1) * SPAN / 4; ++q)
                        part = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], bv[q], part, 0, 0, 0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[rb][q] += (double)part[q];
                }
            }
        }
    }
}

// The tile's pixels, each written once.
__device__ __forceinline__ void put_tile(const FrameDev &F, int X0, int Y0, int wv, int l16, int lg,
                                         const double (*acc)[4])
{
    const int gx = X0 + 16 * wv + l16;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int gy = Y0 + 16 * rb + 4 * lg + q;
            if (gx < F.nx && gy < F.ny)
                ((float *)F.out)[(size_t)gy * F.nx + gx] = (float)acc[rb][q];
        }
}

}  // namespace e2e
