// Photon-noise streams (Sec. 2.2): Philox-4x32-10 (Salmon, Moraes, Dror,
// Shaw, SC'11) with key = seed and counter = (pixel lo, pixel hi, frame
// index, draw block), and the Poisson sampler drawn from it -- Knuth's
// multiplication method (TAOCP vol. 2, 3.4.1) below a mean of 10, Hormann's
// PTRS transformed rejection (Insurance: Math. & Econ. 12, 1993) above.
// Shared by the noise and detector kernels.
#pragma once

#include "dev_common.h"

namespace e2e {

struct Stream {
    uint32_t k0, k1;
    uint32_t c0, c1, c2, c3;
    uint32_t b0, b1, b2, b3;
    int have;
};

// One 32 x 32 -> 64-bit product per multiplier (v_mad_u64_u32) and one
// three-input xor per word: 40 instructions of ten rounds where separate low
// and high products and two-input xors take 80.
__device__ __forceinline__ void philox10(uint32_t &x0, uint32_t &x1, uint32_t &x2, uint32_t &x3,
                                         uint32_t k0, uint32_t k1)
{
    constexpr int kXor3 = 0x96;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)x0 * 0xD2511F53u, p1 = (uint64_t)x2 * 0xCD9E8D57u;
        x0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), x1, k0, kXor3);
        x1 = (uint32_t)p1;
        x2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), x3, k1, kXor3);
        x3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

__device__ __forceinline__ double to_unit(uint32_t a, uint32_t b)
{
    uint64_t m = ((uint64_t)(a >> 5) << 26) | (uint64_t)(b >> 6);
    return ((double)m + 0.5) * (1.0 / 9007199254740992.0);
}

__device__ inline double next_u(Stream &s)
{
    if (s.have == 0) {
        uint32_t x0 = s.c0, x1 = s.c1, x2 = s.c2, x3 = s.c3;
        philox10(x0, x1, x2, x3, s.k0, s.k1);
        s.b0 = x0; s.b1 = x1; s.b2 = x2; s.b3 = x3;
        s.c3 += 1u;
        s.have = 2;
    }
    double u = s.have == 2 ? to_unit(s.b0, s.b1) : to_unit(s.b2, s.b3);
    s.have -= 1;
    return u;
}

// log(k!) for integer k >= 0: exact factorials (all below 2^53) up to 15,
// then Stirling's series for log Gamma(z), z = k + 1 >= 16, through the
// z^-9 term (the first omitted term is below 1.2e-16); within a few ulps of
// the exact value.
__device__ __forceinline__ double log_factorial(double k)
{
    if (k < 16.0) {
        double f = 1.0;
        for (double m = 2.0; m <= k; m += 1.0) f *= m;
        return log(f);
    }
    const double z = k + 1.0, r = 1.0 / z, r2 = r * r;
    double t = 1.0 / 1188.0;
    t = fma(t, r2, -1.0 / 1680.0);
    t = fma(t, r2, 1.0 / 1260.0);
    t = fma(t, r2, -1.0 / 360.0);
    t = fma(t, r2, 1.0 / 12.0);
    return (z - 0.5) * log(z) - z + 0.91893853320467274178 + t * r;
}

// Poisson draw of mean `mean` from the stream: multiplication of uniforms
// below 10, the transformed rejection with squeeze of Hormann (1993, PTRS)
// above.  The acceptance test is the one of the method, evaluated as
// log(V alpha^-1 / (a / us^2 + b)) against k log(mean) - mean - log(k!),
// with log(k!) from log_factorial(); decisions differ from a plain lgamma
// evaluation only when the two sides agree to a few ulps.
__device__ inline double poisson(double mean, Stream &st)
{
    if (!(mean > 0.0)) return 0.0;
    if (mean < 10.0) {
        double L = exp(-mean), prod = next_u(st), k = 0.0;
        for (int guard = 0; prod > L && guard < 100000; ++guard) {
            k += 1.0;
            prod *= next_u(st);
        }
        return k;
    }
    double slam = sqrt(mean), loglam = log(mean);
    double b = 0.931 + 2.53 * slam;
    double a = -0.059 + 0.02483 * b;
    double invalpha = 1.1239 + 1.1328 / (b - 3.4);
    double vr = 0.9277 - 3.6224 / (b - 2.0);
    double k = floor(mean);
    for (int guard = 0; guard < 100000; ++guard) {
        double U = next_u(st) - 0.5;
        double V = next_u(st);
        double us = 0.5 - fabs(U);
        k = floor((2.0 * a / us + b) * U + mean + 0.43);
        if (us >= 0.07 && V <= vr) return k;
        if (k < 0.0 || (us < 0.013 && V > us)) continue;
        if (log(V * invalpha / (a / (us * us) + b)) <= -mean + k * loglam - log_factorial(k))
            return k;
    }
    return k;
}

__device__ __forceinline__ Stream make_stream(uint64_t seed, uint32_t frame, uint64_t p)
{
    Stream s;
    s.k0 = (uint32_t)seed;
    s.k1 = (uint32_t)(seed >> 32);
    s.c0 = (uint32_t)p;
    s.c1 = (uint32_t)(p >> 32);
    s.c2 = frame;
    s.c3 = 0u;
    s.have = 0;
    return s;
}

// num / den for normal positive den: the hardware reciprocal, two Newton steps
// and one correction of the quotient by its exact remainder, which rounds it
// as a division does.
__device__ __forceinline__ double quotient(double num, double den)
{
    double r = __builtin_amdgcn_rcp(den);
    r = fma(r, fma(-den, r, 1.0), r);
    r = fma(r, fma(-den, r, 1.0), r);
    const double q = num * r;
    return fma(fma(-den, q, num), r, q);
}

// Trial `block` of the transformed rejection of a mean >= 10 (uniforms of that
// draw block): 1 accepted by the squeeze or, if FULL, by the acceptance test,
// 0 not (yet).  The same arithmetic as poisson(); the squeeze V <= vr is
// compared as V (b - 2) <= 0.9277 (b - 2) - 3.6224, without the division.
template <bool FULL>
__device__ __forceinline__ bool poisson_trial(double mean, uint64_t seed, uint32_t frame, uint64_t p,
                                              uint32_t block, double *k_out)
{
    uint32_t x0 = (uint32_t)p, x1 = (uint32_t)(p >> 32), x2 = frame, x3 = block;
    philox10(x0, x1, x2, x3, (uint32_t)seed, (uint32_t)(seed >> 32));
    const double slam = sqrt(mean);
    const double b = 0.931 + 2.53 * slam;
    const double a = -0.059 + 0.02483 * b;
    const double U = to_unit(x0, x1) - 0.5, V = to_unit(x2, x3);
    const double us = 0.5 - fabs(U);
    const double k = floor((quotient(2.0 * a, us) + b) * U + mean + 0.43);
    *k_out = k;
    const double b2 = b - 2.0;
    if (us >= 0.07 && V * b2 <= fma(0.9277, b2, -3.6224)) return true;
    if (!FULL || k < 0.0 || (us < 0.013 && V > us)) return false;
    const double invalpha = 1.1239 + 1.1328 / (b - 3.4);
    return log(V * invalpha / (a / (us * us) + b)) <= -mean + k * log(mean) - log_factorial(k);
}

// Poisson draws of the n <= CAP pixels c = 0 .. n - 1 of a workgroup of 256:
// mean_of(c), the pixel's counter pixel_of(c), put(c, draw).  A draw is a pure
// function of (seed, frame, pixel), the one of poisson().
//
// A wave used to run every pixel until its slowest lane was accepted: about
// 2.5 trials, and the acceptance test with its three logarithms in almost every
// wave, though the squeeze settles four pixels of five in the first trial.
// Here the first trials run with the squeeze alone; the pixels it leaves are
// listed in LDS and go on densely packed, trial by trial (a fifth of the
// pixels in the first turn, a third of those in the next), means below 10 (and
// means beyond the trial's range) in a list of their own.
template <int CAP>
struct PoissonLists {
    unsigned short q[2][CAP];   // pixels going on; [0] also holds the small means from its end
    int n[3], small;            // their counts by turn (mod 3), and of the small means
};

template <int CAP, typename Mean, typename Pixel, typename Put>
__device__ __forceinline__ void poisson_span(int n, uint64_t seed, uint32_t frame, Mean mean_of,
                                             Pixel pixel_of, Put put, PoissonLists<CAP> &L)
{
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 3) L.n[tid] = 0;
    if (tid == 3) L.small = 0;
    __syncthreads();
    // appends the lanes with `on` to a list through one LDS add per wave
    auto push = [&](bool on, int *count) -> int {
        const unsigned long long m = __ballot(on);
        if (m == 0) return 0;
        int at = 0;
        const int leader = __ffsll((long long)m) - 1;
        if (lane == leader) at = atomicAdd(count, __popcll(m));
        at = __builtin_amdgcn_readlane(at, leader);
        return at + __popcll(m & ((1ull << lane) - 1ull));
    };
    for (int c0 = 0; c0 < n; c0 += 256) {
        const int c = c0 + tid;
        bool go_on = false, small = false;
        if (c < n) {
            const double mean = mean_of(c);
            if (!(mean > 0.0)) {
                put(c, 0.0);
            } else if (mean < 10.0 || mean > 1e12) {
                small = true;
            } else {
                double k;
                if (poisson_trial<false>(mean, seed, frame, pixel_of(c), 0u, &k)) put(c, k);
                else go_on = true;
            }
        }
        const int i = push(go_on, &L.n[0]);
        if (go_on) L.q[0][i] = (unsigned short)c;
        const int j = push(small, &L.small);
        if (small) L.q[0][CAP - 1 - j] = (unsigned short)c;
    }
    __syncthreads();
    for (int j = tid, m = L.small; j < m; j += 256) {
        const int c = L.q[0][CAP - 1 - j];
        Stream st = make_stream(seed, frame, pixel_of(c));
        put(c, poisson(mean_of(c), st));
    }
    // turn t: trial t of the pixels listed (trial 0 again with the full test);
    // the last few go on in one wave without barriers
    for (uint32_t t = 0; t < 100000u; ++t) {
        const int m = L.n[t % 3];
        if (m == 0) break;
        const unsigned short *from = L.q[t & 1];
        if (m <= 64) {
            if (tid < m) {
                const int c = from[tid];
                const double mean = mean_of(c);
                double k = 0.0;
                for (uint32_t u = t; u < 100000u; ++u)
                    if (poisson_trial<true>(mean, seed, frame, pixel_of(c), u, &k)) break;
                put(c, k);
            }
            break;
        }
        unsigned short *to = L.q[(t + 1) & 1];
        for (int c0 = 0; c0 < m; c0 += 256) {
            const int e = c0 + tid;
            bool go_on = false;
            int c = 0;
            if (e < m) {
                c = from[e];
                double k;
                if (poisson_trial<true>(mean_of(c), seed, frame, pixel_of(c), t, &k)) put(c, k);
                else go_on = true;
            }
            const int i = push(go_on, &L.n[(t + 1) % 3]);
            if (go_on) to[i] = (unsigned short)c;
        }
        // the count after next is read by nobody now
        if (tid == 0) L.n[(t + 2) % 3] = 0;
        __syncthreads();
    }
}

// 53-bit uniform pair of draw block `block` of a pixel's stream (a block
// index the Poisson draws of that pixel never reach when >= 2^31).
__device__ __forceinline__ void uniform_pair(uint64_t seed, uint32_t frame, uint64_t p,
                                             uint32_t block, double *u1, double *u2)
{
    uint32_t x0 = (uint32_t)p, x1 = (uint32_t)(p >> 32), x2 = frame, x3 = block;
    philox10(x0, x1, x2, x3, (uint32_t)seed, (uint32_t)(seed >> 32));
    *u1 = to_unit(x0, x1);
    *u2 = to_unit(x2, x3);
}

}  // namespace e2e
