// Jumps over many power-iteration steps of a level at once.
//
// The iterate after K steps of B = gI - L is, up to its norm, (B/g)^K v.
// With A = I - 2L/g (spectrum in [-1, 1]) B/g = (I + A)/2 and
//   ((1 + y)/2)^K = sum_j c_j T_j(y),  c_0 = C(2K, K)/4^K,
//   c_j = 2 C(2K, K + j)/4^K,  c_{j+1}/c_j = (K - j)/(K + j + 1)
// (Chebyshev polynomials T_j; the expansion of cos^{2K} in cosines of
// multiples of the angle).  The c_j are positive and fall off like
// exp(-j^2/K), so d = 6.2 sqrt(K) products with A give (B/g)^K v to 2e-18
// of ||v||: 199 products in place of 1024 steps.  The sum is stable: every
// T_j(A) has norm 1 and all coefficients are positive.
//
// Algorithm 3 stops at the first step whose (u, v) reaches 1 - tol, so a
// jump may only cross steps that would not have stopped.  The products
// give the Chebyshev moments mu_{2j} = 2 (T_j v, T_j v) - mu_0 and
// mu_{2j+1} = 2 (T_j v, T_{j+1} v) - mu_1 up to 2d, hence the power moments
//   m_p = (v, (B/g)^p v) = sum_j c_j^{(p)} mu_j       (p <= 4K)
// and the quantity the test looks at after k steps,
//   (u, v)_k = m_{2k-1} / sqrt(m_{2k-2} m_{2k}),      k <= 2K,
// for steps inside the jump and as many again beyond it.  A jump is kept
// only if 1 - (u, v)_k stays above tol (with a margin) at samples over all
// of its steps; else it is taken back (the start vector is kept) and
// shortened to the last sample before the crossing.  The last steps before
// the test passes are always ordinary steps with the test itself, so the
// step count and the iterate are those of the plain loop (in exact
// arithmetic; the rounding error of a jump is that of a few steps).
#pragma once

#include "cmg_dev.h"

namespace cmg {

// Jumps of fewer steps save too little (100 steps: 63 products).
constexpr int kJumpMinK = 100;
constexpr int kJumpMaxK = 4096;
constexpr int kJumpMaxD = 400;        // products of the longest jump (6.2 sqrt(4096) + 1 = 398)
constexpr int kJumpMoments = 2 * kJumpMaxD + 2;
constexpr int kJumpSamples = 256;     // samples of (u, v)_k over k <= 2K
constexpr int kJumpWords = kJumpMoments + kJumpSamples;  // doubles of a moment buffer
// Plain steps before the first jump of a level and between an estimate and
// the one before it: the fast modes die first, after which the logarithm of
// 1 - (u, v) falls ever more slowly and its slope bounds the steps left
// from below.
constexpr int kJumpPlain = 24;  // a multiple of 8
// A sample this close to the tolerance counts as a crossing.
constexpr double kJumpMargin = 1.02;
// 1 - (u, v) from the moments carries about 1e-13 of absolute error.
constexpr double kJumpTolMin = 1e-10;
// Steps to try where 1 - (u, v) rises.
constexpr double kJumpRising = 512.0;
// ||(B/g)^K v|| may fall to e^-3 within a jump (its error is relative to ||v||).
constexpr double kJumpDecay = 3.0;

// Steps of a jump: at most `want` and `left`, and few enough that the norm
// (||B v|| / g = r on the last plain step) keeps e^-kJumpDecay of itself; 0
// if that is too short (also for a want that is not a number).
__device__ __forceinline__ int jump_steps(double want, double r, int left) {
    if (r < 1.0) want = fmin(want, kJumpDecay / -log(r));
    want = fmin(want, (double)left);
    if (!(want >= (double)kJumpMinK)) return 0;
    return (int)fmin(want, (double)kJumpMaxK);
}

// products of a jump of K steps
__device__ __forceinline__ int jump_products(int K) { return (int)ceil(6.2 * sqrt((double)K)) + 1; }

// Whether the `since`-th plain step is one after which a jump is considered
// (an estimate costs two logarithms and as many divisions, about as much as
// a step of a small level, so one in sixteen).
__device__ __forceinline__ bool jump_due(int since) { return since >= kJumpPlain && (since & 15) == (kJumpPlain & 15); }

// Steps to jump after a plain step with (u, v) = utv (utvp the step before)
// that did not stop; tol < 0: no test, a fixed count.
__device__ __forceinline__ int jump_plan(double utv, double utvp, double tol, double r, int left) {
    if (left < kJumpMinK) return 0;
    double want = (double)left;
    if (tol >= 0.0) {
        const double dl = 1.0 - utv, dp = 1.0 - utvp;
        if (!(dl > tol)) return 0;
        // a level whose 1 - (u, v) rises (the vector turns from one mode to
        // a slower one) is far from its end: a power-law level of 594
        // vertices rose for 1310 of its 2781 steps
        want = dl < dp ? 0.9 * (log(dl / tol) / log(dp / dl)) - 8.0 : kJumpRising;
    }
    return jump_steps(want, r, left);
}

// coefficient of the vector after product j + 1 from that of product j
// (c_1 / c_0 = 2K / (K + 1))
__device__ __forceinline__ double jump_coef(double cj, int K, int j) {
    return cj * ((double)(K - j) / (double)(K + j + 1));
}

// Moments after product j (0 the first) with the sums sxy = (T_j, T_{j+1}),
// syy = (T_{j+1}, T_{j+1}) and, for the first, sxx = (T_0, T_0).
__device__ __forceinline__ void jump_moments(double* mom, int j, double sxy, double syy, double sxx) {
    if (j == 0) {
        mom[0] = sxx;
        mom[1] = sxy;
        mom[2] = 2.0 * syy - sxx;
    } else {
        mom[2 * j + 1] = 2.0 * sxy - mom[1];
        mom[2 * j + 2] = 2.0 * syy - mom[0];
    }
}

// 1/x for positive integers x to double rounding (reciprocal estimate and
// two Newton steps; a division would cost several times that)
__device__ __forceinline__ double jump_rcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

// 1 - (u, v)_k from the moments mom[0 .. nm-1].  The three sums run
// together; c_0^{(p)} / c_0^{(p-1)} = (2p - 1)/(2p) is taken out of them.
__device__ __forceinline__ double jump_delta(const double* mom, int nm, int k) {
    const double p = (double)(2 * k - 2);
    const int jm = min(2 * k, nm - 1);
    double a = mom[0], b = a, c = a;
    double ca = 2.0, cb = 2.0, cc = 2.0;
    double r0 = jump_rcp(p + 1.0), r1 = jump_rcp(p + 2.0);
    for (int j = 0; j < jm; ++j) {
        const double x = (double)j;
        const double r2 = jump_rcp(p + x + 3.0);
        ca *= (p - x) * r0;
        cb *= (p + 1.0 - x) * r1;
        cc *= (p + 2.0 - x) * r2;
        r0 = r1;
        r1 = r2;
        const double m = mom[j + 1];
        a = fma(ca, m, a);
        b = fma(cb, m, b);
        c = fma(cc, m, c);
    }
    const double q = 4.0 * (double)k;
    const double rho2 = (q - 3.0) / (q - 2.0) * (q / (q - 1.0)) * (b * b) / (a * c);
    return (1.0 - rho2) / (1.0 + sqrt(rho2));
}

// step of sample s of ns over the 2K steps that the moments reach
__device__ __forceinline__ int jump_sample(int s, int ns, int K) {
    return (int)(((long long)(s + 1) * 2 * K + ns - 1) / ns);
}

// From the samples dl[0 .. ns-1] (one wavefront, all lanes): *safe = the
// steps that do not pass the test (2K if none of the samples does), *next =
// what can be jumped after the K steps (an estimate beyond the samples).
__device__ __forceinline__ void jump_judge(const double* dl, int ns, int K, double tol, int* safe, int* next) {
    const int lane = (int)threadIdx.x & 63;
    int first = ns;
    for (int s = lane; s < ns; s += 64)
        if (!(dl[s] >= kJumpMargin * tol)) first = min(first, s);
    for (int o = 32; o > 0; o >>= 1) first = min(first, __shfl_xor(first, o, kWave));
    if (first < ns) {
        *safe = first > 0 ? jump_sample(first - 1, ns, K) : 0;
        *next = *safe - K;
        return;
    }
    *safe = 2 * K;
    const int s1 = ns - 1, s0 = ns - 1 - ns / 16;
    const double d0 = dl[s0], d1 = dl[s1];
    double more = d1 < d0 ? (double)kJumpMaxK : 2.0 * (double)K;
    if (d1 < d0 && d1 > tol)
        more = 0.9 * (log(d1 / tol) / log(d0 / d1)) * (double)(jump_sample(s1, ns, K) - jump_sample(s0, ns, K));
    *next = K + (int)fmin(more, (double)kJumpMaxK);
}

// After a jump of K steps: true if it is kept.  *more: steps to try to jump
// next; *hold: else plain steps before the next estimate.
__device__ __forceinline__ bool jump_verdict(int K, int safe, int next, bool fixed, int* more, int* hold) {
    const bool keep = fixed || safe >= K;
    const int n = fixed ? 0 : keep ? next : safe;
    *more = n >= kJumpMinK ? n : 0;
    *hold = n >= kJumpMinK ? 0 : max(n, 0);
    return keep;
}

}  // namespace cmg
