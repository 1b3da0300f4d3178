// bdc_device.h -- device arithmetic of the gfx950 sampler: counter-based random
// numbers and the per-pixel likelihood of the paper's camera model.
//
// Pixel model (Methods, Eqs. 3-6):  with c = (w - o)/G and a = G^2/(2 sigma^2),
//   L(mu) = (2 pi sigma^2)^-1/2 * sum_{k>=0} exp(-a (k - c)^2) mu^k e^-mu / k!.
// Summands are log-concave in k.  Their ratio r_k = W_{k+1}/W_k =
// mu exp(-a (2k + 1 - 2c)) / (k + 1) is a geometric sequence in exp(2a) times
// 1/(k+1), which is what the inner loops below iterate.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bdc_consts.h"

namespace bdc {

// ---------------------------------------------------------------------------
// Counter-based generator: Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11).
// Ten rounds of two 32x32->64 multiplies with a Weyl-sequence key schedule.
// ---------------------------------------------------------------------------
__host__ __device__ inline uint4 philox4x32_10(uint4 ctr, uint2 key) {
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * ctr.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * ctr.z;
        const uint32_t h0 = (uint32_t)(p0 >> 32), l0 = (uint32_t)p0;
        const uint32_t h1 = (uint32_t)(p1 >> 32), l1 = (uint32_t)p1;
        ctr = make_uint4(h1 ^ ctr.y ^ key.x, l1, h0 ^ ctr.w ^ key.y, l0);
        key.x += 0x9E3779B9u;
        key.y += 0xBB67AE85u;
    }
    return ctr;
}

// Random-number streams of one (pixel, sweep, chain) counter.
enum : uint32_t { STREAM_PROPOSAL = 0, STREAM_ACCEPT = 1, STREAM_INIT = 2, STREAM_BLOCK = 3, STREAM_BLOCK_ACCEPT = 4 };

__device__ inline uint4 draw(uint2 key, uint32_t pixel, uint32_t sweep, uint32_t chain, uint32_t stream) {
    return philox4x32_10(make_uint4(pixel, sweep, chain, stream), key);
}

// Open-interval uniform from the top 23 bits: ((x >> 9) + 1/2) 2^-23, exact in FP32.
__device__ inline float u01(uint32_t x) { return ((float)(x >> 9) + 0.5f) * (1.0f / 8388608.0f); }

// Box-Muller from words 0 and 1 of one block (cosine branch).
__device__ inline float box_muller(uint4 r) {
    const float u1 = u01(r.x), u2 = u01(r.y);
    return sqrtf(-2.0f * logf(u1)) * cospif(2.0f * u2);
}

// ---------------------------------------------------------------------------
// Constants of the phi window and the ratio recurrence.
// ---------------------------------------------------------------------------
// Above this a the geometric factor exp(2a) leaves FP32 range: those pixels
// (read noise far below one photon) take a short direct-exponent loop.
constexpr float A_RECUR_MAX = 40.0f;
// Depth of the phi window: every omitted summand is below the largest by
// exp(-TAIL_T) at least (log-concavity bound), total < 1e-8 relative.
constexpr float TAIL_T = 20.0f;

// Per-pixel constants of one footprint evaluation.  Stored per pixel (one
// 16-byte record, derived once per frame): c, 2a, and L0 = 2a(c - ks) -
// log(ks + 1), iB = 1/(2a + 1/(ks + 1)) with ks = max(c, 0), so that the
// tangent step of L (below) at ks is ks + (L0 + log mu) iB.  Derived in
// registers at load: ks, 1/(2a) and h0 = sqrt(TAIL_T / a), the half-width
// bound from the curvature 2a.  (16 bytes keep a workgroup's footprint of
// records small enough for the resident workgroups of an XCD to share its L2.)
struct PixConst {
    float c, a2, inv2a;
    float ks, L0, iB, h0;
};

// Sums that are rounded by themselves.  The compiler may fuse a product into a
// sum or not, differently in each kernel and version of the source; where a
// chain's state or decision depends on it, the code says which (these or fmaf),
// so that the same inputs give the same chain.
__device__ inline float add_rn(float a, float b) {
#pragma clang fp contract(off)
    return a + b;
}
__device__ inline float mul_rn(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}

__device__ inline float fast_ln(float x) { return __builtin_amdgcn_logf(x) * 0.69314718055994531f; }
__device__ inline float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// log(1 + x) to a few ulp.  |x| < 1/16: the Taylor series through x^8
// (remainder below x^9/9, < 3e-11 relative).  Otherwise the hardware log of
// u = fl(1 + x) with Kahan's correction log1p(x) = log(u) x / (u - 1), which
// cancels the rounding of u; there |log u| > 0.06, where the hardware log's
// error is a few ulp of the result.
__device__ inline float log1p_k(float x) {
    float s = fmaf(x, -0.125f, 0.14285714285714285f);
    s = fmaf(x, s, -0.16666666666666666f);
    s = fmaf(x, s, 0.2f);
    s = fmaf(x, s, -0.25f);
    s = fmaf(x, s, 0.33333333333333333f);
    s = fmaf(x, s, -0.5f);
    s = fmaf(x, s, 1.0f);
    const float series = x * s;
    const float u = 1.0f + x;
    const float kahan = fast_ln(u) * (x * fast_rcp(u - 1.0f));
    return fabsf(x) < 0.0625f ? series : kahan;
}

// exp(y) in double with FP32 relative accuracy over the whole double range:
// 2^(y log2 e) = 2^n * 2^f, f in [0, 1) through the FP32 exp2.
__device__ inline double exp_wide(double y) {
    const double z = y * 1.4426950408889634;
    const double n = floor(z);
    const float f = (float)(z - n);
    return ldexp((double)__builtin_amdgcn_exp2f(f), (int)fmax(fmin(n, 2000.0), -2000.0));
}

// The same for |y| < 2^30 (no clamp of the exponent; ldexp saturates).
__device__ inline double exp_wide_b(double y) {
    const double z = y * 1.4426950408889634;
    const double n = floor(z);
    const float f = (float)(z - n);
    return ldexp((double)__builtin_amdgcn_exp2f(f), (int)n);
}

// exp(y) for 0 < y <= 2 A_RECUR_MAX in FP32 range, FP32 relative accuracy.
__device__ inline double exp_small(float y) {
    const double z = (double)y * 1.4426950408889634;
    const double n = floor(z);
    const float f = (float)(z - n);
    return (double)__builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// The 2a that a pixel's record holds.  The recurrences step by exp_small(2a), whose
// rounding is another 2a, off by up to 6e-8: over a window of n terms that moves a
// mean count's change by up to n 6e-8 of it, and by another amount in another window.
// Below WIDE_A2 (read noise above ten photons, windows of hundreds of terms) the
// record therefore holds the logarithm of that step, so that every evaluation of the
// pixel agrees on its read noise, which is off by 3e-6 of itself at 10 photons and by
// 3e-4 at 100.
constexpr float WIDE_A2 = 0.01f;
__device__ inline float record_a2(float a2) {
    const double q = exp_small(a2);
    return a2 < WIDE_A2 && q > 1.0 ? (float)log(q) : a2;
}

// 1/n, 1/(n-1), 1/(n-2), 1/(n-3) for 4 <= n < 2^20 from one hardware
// reciprocal of their product and one Newton step: each reciprocal is the
// product of the other three factors with it (relative error below 1e-15).
__device__ inline void recip4(int n, double cv[4]) {
    const double na = (double)n, nb = na - 1.0, nc = na - 2.0, nd = na - 3.0;
    const double pab = na * nb, pcd = nc * nd, P = pab * pcd;
    double R = __builtin_amdgcn_rcp(P);
    R = fma(R, fma(-P, R, 1.0), R);
    const double Rab = R * pab, Rcd = R * pcd;
    cv[0] = nb * Rcd;
    cv[1] = na * Rcd;
    cv[2] = nd * Rab;
    cv[3] = nc * Rab;
}

// 1/x: the hardware reciprocal (about 27 bits) and one Newton step; rcp_nr2: two
// steps, full double accuracy.
__device__ inline double rcp_nr(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    return r * fma(-x, r, 2.0);
}

__device__ inline double rcp_nr2(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// ---------------------------------------------------------------------------
// phi window.  For mean mu the log-summand f(k) = -a (k-c)^2 + k log mu - lgamma(k+1)
// is concave with f'' <= -(2a + 1/(k+1)).  Its continuous mode k* lies where
//   2a(c - k) + log mu - digamma(k + 1) = 0,  and log(k+1/2) < digamma(k+1) < log(k+1).
// Lower bound: L(k) = 2a(c - k) + log mu - log(k + 1) is convex and decreasing
// with L(k*) >= 0, so one tangent (Newton) step from any point lands at or below
// its root, hence below k*.  Upper bound: for k >= p, log(k + 1/2) >= log(p + 1/2)
// so f'(k) < 2a(c - k) + log mu - log(p + 1/2) <= 0 once k >= c + log(mu/(p+1/2))/(2a).
// The window is [p - h, q + h] with h^2 = 2 TAIL_T / kappa, kappa a lower bound on
// the curvature: 2a, and 1/(2q + 4T + 2) (h <= q + 4T + 1).  mu enters
// monotonically, so the window of [mu_lo, mu_hi] covers both the current and
// the proposed mean.
// ---------------------------------------------------------------------------
struct Window { int lo, hi; bool ok; };

__device__ inline Window finish_window(float p, float q, float h0) {
    // hardware square root: the half-width only needs a few significant digits
    const float hp = __builtin_amdgcn_sqrtf(2.0f * TAIL_T * (2.0f * q + 4.0f * TAIL_T + 2.0f));
    const float h = fminf(h0, hp);
    Window w;
    // photon counts beyond 2^20 per pixel are outside the model's working range
    // (and would make the loops unbounded): flagged, the caller rejects
    w.ok = (q + h < 1048576.0f);
    w.lo = w.ok ? (int)fmaxf(floorf(p - h), 0.0f) : 0;
    w.hi = w.ok ? (int)ceilf(q + h) : 0;
    return w;
}

// Newton refinement of the lower bound (slow path for a loose bracket); the
// bracket travels in registers (by value), so the common path touches no
// private memory.
__device__ __noinline__ float2 refine_bracket(float lmu_lo, float lmu_hi, PixConst pc, float2 pq) {
    float p = pq.x, q = pq.y;
    for (int it = 0; it < 8 && q - p > 6.0f; ++it) {
        const float k1 = p + 1.0f;
        const float L = pc.a2 * (pc.c - p) + lmu_lo - fast_ln(k1);
        const float pn = fmaxf(fmaf(L * k1, fast_rcp(fmaf(pc.a2, k1, 1.0f)), p), 0.0f);
        if (pn - p < 0.25f) break;
        p = pn;
        q = fmaxf(p, pc.c + (lmu_hi - fast_ln(p + 0.5f)) * pc.inv2a);
    }
    return make_float2(p, q);
}

__device__ inline Window phi_window(float lmu_lo, float lmu_hi, const PixConst& pc) {
    float2 pq;
    pq.x = fmaxf(fmaf(pc.L0 + lmu_lo, pc.iB, pc.ks), 0.0f);
    pq.y = fmaxf(pq.x, pc.c + (lmu_hi - fast_ln(pq.x + 0.5f)) * pc.inv2a);
    if (pq.y - pq.x > 6.0f) pq = refine_bracket(lmu_lo, lmu_hi, pc, pq);
    return finish_window(pq.x, pq.y, pc.h0);
}

// log(num / den) for positive double sums, to FP32 relative accuracy of the
// result at every scale, in one branch-free path: the ratio's binary exponent
// is split off in double with the mantissa m scaled into [sqrt(1/2), sqrt(2)),
// and log m = 2 atanh(z), z = (m - 1)/(m + 1), |z| <= 0.1716, by its odd
// series through z^9 (remainder below 5e-9 relative).  m - 1 is exact in
// double, so ratios near 1 keep their small logarithm to full relative
// accuracy, and ratios far from 1 (a proposal far from the current state)
// never round against 1.
__device__ inline double log_ratio(double num, double den) {
    const double q = num * __builtin_amdgcn_rcp(den);
    int e = __builtin_amdgcn_frexp_exp(q);
    double m = __builtin_amdgcn_frexp_mant(q);           // [1/2, 1)
    if (m < 0.70710678118654752) { m += m; e -= 1; }     // [sqrt(1/2), sqrt(2))
    const float z = (float)((m - 1.0) * __builtin_amdgcn_rcp(m + 1.0));
    const float z2 = z * z;
    float poly = fmaf(z2, 0.22222222222222222f, 0.28571428571428571f);
    poly = fmaf(z2, poly, 0.4f);
    poly = fmaf(z2, poly, 0.66666666666666667f);
    poly = fmaf(z2, poly, 2.0f);
    return fma((double)e, 0.69314718055994531, (double)(z * poly));
}

// ---------------------------------------------------------------------------
// Sharp read noise (a > A_RECUR_MAX): the window holds a handful of terms; each
// log-summand relative to the one at k0 is formed directly,
//   lw_k = -a((k-c)^2 - (k0-c)^2) + (k - k0) log mu - sum_{j in (k0, k]} log j,
// and both sums are max-free (every lw_k <= ~0 near the mode).
// ---------------------------------------------------------------------------
__device__ inline double lgamma_diff(int k, int k0) {   // lgamma(k+1) - lgamma(k0+1)
    double s = 0.0;
    if (k > k0) for (int j = k0 + 1; j <= k; ++j) s += log((double)j);
    else for (int j = k + 1; j <= k0; ++j) s -= log((double)j);
    return s;
}

__device__ inline double delta_ell_sharp(float d, float lmu, float lx, Window win, float cf, float a2) {
    int k0 = (int)rintf(fmaxf(cf, 0.0f));
    k0 = k0 < win.lo ? win.lo : (k0 > win.hi ? win.hi : k0);
    const double a = 0.5 * (double)a2, c = cf, lmd = (double)lmu;
    double s0 = 0.0, s1 = 0.0;
    for (int k = win.lo; k <= win.hi; ++k) {
        const double lw = -a * ((k - c) * (k - c) - (k0 - c) * (k0 - c)) + (k - k0) * lmd - lgamma_diff(k, k0);
        s0 += exp_wide(lw);
        s1 += exp_wide(lw + (k - k0) * (double)lx);
    }
    return -(double)d + (double)k0 * (double)lx + log_ratio(s1, s0);
}

// ---------------------------------------------------------------------------
// Long windows.  The sums of the recurrences below are relative to the window's
// lowest weight, which a mode hundreds of counts above it takes out of the double
// range (a = 0.00317, c = 482, mu 480 -> 11: the value is -595, an overflowed sum gave
// +359).  Windows of more than LONG_WINDOW terms and sums beyond SUM_MAX are taken
// here, with sums scaled down as they grow and, since they are long, exp(2a) in double.
// ---------------------------------------------------------------------------
constexpr int LONG_WINDOW = 128;
constexpr double SUM_MAX = 1e300;

// log(sum_k W_k x^k / sum_k W_k) - d over the window.
__device__ inline double delta_ell_long(float mu, float d, Window win, float c, float a2) {
    const double m = (double)mu, x = 1.0 + (double)d / m, qi = exp((double)a2);
    double G = m * exp(-(double)a2 * ((double)win.hi - 0.5 - (double)c));
    double acc0 = 0.0, acc1 = 0.0, one0 = 1.0, one1 = 1.0;          // sums and the lowest weight, times 2^-e
    int e = 0;                                                      // e1 - e0
#pragma unroll 1
    for (int n = win.hi; n > win.lo; --n) {
        const double r = G * rcp_nr2((double)n);
        G *= qi;
        acc0 = r * (acc0 + one0);
        acc1 = r * x * (acc1 + one1);
        if (acc0 > 0x1p500) {
            acc0 *= 0x1p-500;
            one0 *= 0x1p-500;
            e -= 500;
        }
        if (acc1 > 0x1p500) {
            acc1 *= 0x1p-500;
            one1 *= 0x1p-500;
            e += 500;
        }
    }
    return log((one1 + acc1) / (one0 + acc0)) + (double)e * 0.69314718055994531 + (double)win.lo * log(x) - (double)d;
}

// What the recurrences do not take.  (One call for all: a call site costs its kernel
// registers.)
__device__ __noinline__ double delta_ell_rare(float mu, float d, float lmu, float lx, Window win, float c, float a2) {
    return a2 > 2.0f * A_RECUR_MAX ? delta_ell_sharp(d, lmu, lx, win, c, a2) : delta_ell_long(mu, d, win, c, a2);
}

// ---------------------------------------------------------------------------
// Local series of one pixel's log-likelihood (used by the block-series scan).
// With v = y/mu, ell(mu + y) - ell(mu) = -y + log E_mu[(1 + v)^phi], the
// expectation under the photon-count posterior at mu.  As a function of mu the
// pixel factor sum_k exp(-a(k - c)^2) mu^k / k! is exp(-a c^2) times the image
// of exp(z), z = mu exp(2ac), under the multiplier sequence exp(-a k^2)
// (Laguerre); by the Polya-Schur theorem it has only real negative zeros, so
//   log E[(1 + v)^phi] = sum_i log(1 + beta_i v),   0 < beta_i < 1,
// and its Taylor coefficients h_j = (-1)^(j+1) sum_i beta_i^j / j give, after
// order J, a remainder of at most  s2 |v|^(J+1) / ((J + 1)(1 - |v|))  with
// s2 = sum_i beta_i^2 = E[phi] - Var[phi] = -2 h_2.
//
// series_at() evaluates h_1..h_4 at mu exactly (up to rounding) from the same
// phi window as delta_ell: Horner's rule from the window top on the degree-4
// polynomial S(v) = sum_k (W_k / W_lo)(1 + v)^(k - lo), then the power-series
// logarithm of S(v)/S(0) plus lo log(1 + v).  Returned, in y-units:
//   ell(mu + y) - ell(mu) = b1 y + b2 y^2 + b3 y^3 + b4 y^4,
//   b1 = h1/mu - 1, bj = hj/mu^j,
// and the radius R = u mu, the largest |y| whose bound stays below
// SERIES_TAU / 2 (u <= 1/2, so mu + y > 0 inside it).  R = 0 (never used in
// place of the direct evaluation) for sharp read noise, whose coefficients serve
// the bounds of series_bound only, and, with b2 > 0 (no
// series has it), for an unusable window or mu <= 0.
// ---------------------------------------------------------------------------
constexpr float SERIES_TAU = 3e-9f;

struct Series { float4 b; float R; };
__device__ inline float4 no_series() { return make_float4(0.0f, 1.0f, 0.0f, 0.0f); }

// Series from the coefficients g_j of v^j of the change of log Z.
__device__ inline Series series_of_log(double g1, double g2, double g3, double g4, float mu) {
    Series out;
    const double im = rcp_nr2((double)mu), im2 = im * im;
    out.b = make_float4((float)(g1 * im - 1.0), (float)(g2 * im2), (float)(g3 * im2 * im), (float)(g4 * im2 * im2));
    // radius: u0 = (tau/2 * 5 / s2)^(1/5) solves s2 u^5 / 5 = tau/2; the factor
    // (1 - u0)^(1/5) makes room for the 1/(1 - u) of the bound; R = 0 where a sum
    // overflowed and the coefficients are no numbers
    const float s2 = (float)(-2.0 * g2), s2v = s2 == s2 ? fmaxf(s2, 1e-30f) : INFINITY;
    float u = __builtin_amdgcn_exp2f(0.2f * __builtin_amdgcn_logf(2.5f * SERIES_TAU * __builtin_amdgcn_rcpf(s2v)));
    u = fminf(u, 0.5f);
    u *= __builtin_amdgcn_exp2f(0.2f * __builtin_amdgcn_logf(1.0f - u));
    out.R = u * mu;
    return out;
}

// Series of the pixel at mean mu from the window polynomial S(v) =
// sum_k (W_k / W_ref)(1 + v)^(k - lo) (coefficients S0, A1..A4).
__device__ inline Series series_finish(double S0, double A1, double A2, double A3, double A4, int lo, float mu) {
    const double iS = rcp_nr2(S0);
    const double s1 = A1 * iS, s2 = A2 * iS, s3 = A3 * iS, s4 = A4 * iS;
    // log(1 + s1 v + s2 v^2 + ...): h_j = s_j - (1/j) sum_{i<j} i h_i s_{j-i}
    const double h1 = s1;
    const double h2 = s2 - 0.5 * h1 * s1;
    const double h3 = s3 - (h1 * s2 + 2.0 * h2 * s1) * (1.0 / 3.0);
    const double h4 = s4 - 0.25 * (h1 * s3 + 2.0 * h2 * s2 + 3.0 * h3 * s1);
    const double L = (double)lo;                     // + lo log(1 + v)
    const double g1 = h1 + L, g2 = h2 - 0.5 * L, g3 = h3 + L * (1.0 / 3.0), g4 = h4 - 0.25 * L;
    return series_of_log(g1, g2, g3, g4, mu);
}

// Sharp read noise (a > A_RECUR_MAX): the few weights of the window relative to
// the one nearest to c, outwards by their ratios; R = 0.
__device__ __noinline__ Series series_sharp(float mu, Window win, float c, float a2) {
    int k0 = (int)rintf(fmaxf(c, 0.0f));
    k0 = k0 < win.lo ? win.lo : (k0 > win.hi ? win.hi : k0);
    double S0 = 0.0, S1 = 0.0, S2 = 0.0, S3 = 0.0, S4 = 0.0;
    auto add = [&](int k, double w) {
        const double n = (double)(k - win.lo);
        S0 += w;
        w *= n;
        S1 += w;
        w *= (n - 1.0) * 0.5;
        S2 += w;
        w *= (n - 2.0) * (1.0 / 3.0);
        S3 += w;
        S4 += w * (n - 3.0) * 0.25;
    };
    auto ratio = [&](int k) { return (double)mu * exp_wide(-(double)a2 * ((double)k + 0.5 - (double)c)); };   // (k + 1) W_(k+1) / W_k
    double w = 1.0;
    add(k0, w);
    for (int k = k0; k < win.hi && w > 1e-30; ++k) {
        w *= ratio(k) * rcp_nr((double)(k + 1));
        add(k + 1, w);
    }
    w = 1.0;
    for (int k = k0 - 1; k >= win.lo && w > 1e-30; --k) {
        w *= (double)(k + 1) * exp_wide((double)a2 * ((double)k + 0.5 - (double)c)) * rcp_nr((double)mu);
        add(k, w);
    }
    Series out = series_finish(S0, S1, S2, S3, S4, win.lo, mu);
    out.R = 0.0f;
    if (!(fabsf(out.b.x) + fabsf(out.b.y) + fabsf(out.b.z) + fabsf(out.b.w) < INFINITY)) out.b = no_series();
    return out;
}

// ---------------------------------------------------------------------------
// EMCCD pixel: photoelectrons phi ~ Poisson(mu), the multiplication register's
// output x ~ Gamma(phi, 1) (photon units) for phi >= 1 and x = 0 for phi = 0,
// reading w = o + G x with read noise on the zero-photon reading.  With
// c = (w - o)/G and A = Normal(w; o, sigma^2),
//   L(mu) = e^-mu [ A + [c > 0] (e^-c / G) sqrt(mu / c) I_1(2 sqrt(mu c)) ]
// (the photoelectron sum in closed form).  Per-pixel record (c, -1, log A,
// -c - log G): the -1 in place of 2a marks the model; -c - log G is -inf for
// c <= 0, where no photoelectron can have been amplified.
// ---------------------------------------------------------------------------
// log I_1(z), z > 0, in double: the power series
//   I_1(z) = sum_k (z/2)^(2k+1) / (k! (k+1)!)
// for z < 24 (summed until a term falls below 1e-17 of the sum), and for
// z >= 24 the asymptotic expansion (Abramowitz & Stegun 9.7.1, order 1)
//   I_1(z) = e^z / sqrt(2 pi z) sum_k a_k,  a_0 = 1,
//   a_k = -a_(k-1) (4 - (2k - 1)^2) / (8 k z),
// whose terms fall over the first 2z of them, truncated below 1e-17.  Both
// run four terms per step with the step's reciprocals formed off the chain of
// products (hardware reciprocal and one Newton step, full double accuracy),
// so the chain is multiplies and adds only; the tolerance is checked once per
// step (the extra terms of the last step only add more of the exact sum).
__device__ inline double log_i1(double z) {
    if (z < 24.0) {
        const double h = 0.5 * z, h2 = h * h;
        double t = h, s = h;
#pragma unroll 1
        for (int k = 0; k < 200; k += 4) {
            double q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = h2 * rcp_nr((double)(k + u + 1) * (double)(k + u + 2));
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                t *= q[u];
                s += t;
            }
            if (t < 1e-17 * s) break;
        }
        return log(s);
    }
    const double iz8 = 0.125 / z;
    double a = 1.0, s = 1.0;
#pragma unroll 1
    for (int k = 1; k < 48; k += 4) {
        double q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double m = (double)(2 * (k + u) - 1);
            q[u] = (m * m - 4.0) * iz8 * rcp_nr((double)(k + u));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a *= q[u];
            s += a;
        }
        if (fabs(a) < 1e-17 * s) break;
    }
    return z - 0.5 * log(6.283185307179586 * z) + log(s);
}

// log(e^a + e^b) for finite a, b that may be -inf.
__device__ inline double lse2(double a, double b) {
    const double m = fmax(a, b);
    return m + log1p(exp(-fabs(a - b)));
}

// log L(mu) + mu of an EMCCD pixel from its record fields: log A and
// lB = -c - log G, mu > 0.
__device__ inline double emccd_lse(double mu, double c, double lA, double lB) {
    if (!(c > 0.0)) return lA;
    return lse2(lA, lB + 0.5 * log(mu / c) + log_i1(2.0 * sqrt(mu * c)));
}

// ell(mu + d) - ell(mu) of an EMCCD pixel (NaN when mu + d <= 0).
__device__ inline double delta_ell_emccd(float mu, float d, const PixConst& pc) {
    const double m0 = (double)mu, m1 = (double)mu + (double)d;
    if (!(m1 > 0.0) || !(m0 > 0.0)) return __builtin_nan("");
    if (d == 0.0f) return 0.0;
    if (!(pc.c > 0.0f)) return -(double)d;
    return (emccd_lse(m1, pc.c, pc.L0, pc.iB) - emccd_lse(m0, pc.c, pc.L0, pc.iB)) - (double)d;
}

// ---------------------------------------------------------------------------
// Likelihood change of one footprint pixel:
//   ell(mu + d) - ell(mu) = -d + log( sum_k W_k x^k / sum_k W_k ),  x = 1 + d/mu,
// i.e. the log of the mean of x^phi under the photon-count posterior at mu.
// Both sums run over one window by Horner's rule from the top (normalised at
// the window's lower end, so x^k -> x^(k - lo)), in double precision:
//   acc0 <- r_k (1 + acc0),  acc1 <- x r_k (1 + acc1),  r_k = G_k / (k + 1),
//   G_k = mu exp(-a(2k + 1 - 2c)),  G_{k-1} = G_k exp(2a).
// For a <= A_RECUR_MAX and a short window the summands span less than the double
// range (TAIL_T nats deep plus a bracket of a few photons); delta_ell_rare takes the
// others.  Returns NaN when mu + d <= 0 and for counts beyond the window's range
// (the caller then rejects).  inv_tab[k] = 1/k for k < INV_TABLE.
// ---------------------------------------------------------------------------
// TABLE: 1/(k+1) from inv_tab (staged in LDS by the caller), else computed
// (recip4), which keeps memory latency out of the recurrence when no table
// fits in LDS.
template <bool TABLE>
__device__ inline double delta_ell_t(float mu, float d, const PixConst& pc, const double* inv_tab, int& nterms) {
    const float mu1 = mu + d;
    if (!(mu1 > 0.0f) || !(mu > 0.0f)) return __builtin_nan("");
    if (d == 0.0f) return 0.0;
    const float t = d * fast_rcp(mu);             // relative change
    const float lx = log1p_k(t);                  // log x
    const float lmu = fast_ln(mu);
    const Window win = phi_window(lmu + fminf(lx, 0.0f), lmu + fmaxf(lx, 0.0f), pc);
    if (!win.ok) return __builtin_nan("");
    nterms += win.hi - win.lo + 1;                // the window's terms (work measure)
    // The recurrence runs in steps of four terms: the window is widened to a
    // multiple of four (downwards while that stays >= 0, else upwards).  Extra
    // summands only add more of the exact sum.
    int lo = win.lo, hi = win.hi;
    const int n4 = (hi - lo + 3) & ~3;
    lo = hi - n4;
    if (lo < 0) { hi -= lo; lo = 0; }
    const double x = 1.0 + (double)t;
    const double qi = exp_small(pc.a2);           // exp(2a), the ratio of successive G
    const int k_top = hi - 1;
    // |exponent| <= 2 A_RECUR_MAX (2^20 + 1): within exp_wide_b's range
    double G = (double)mu * exp_wide_b(-(double)pc.a2 * ((double)k_top + 0.5 - (double)pc.c));
    double acc0 = 0.0, acc1 = 0.0;
    const bool rare = pc.a2 > 2.0f * A_RECUR_MAX || win.hi - win.lo > LONG_WINDOW;
    if (rare) {
    } else if (!TABLE || hi < INV_TABLE) {
        const double* iv = inv_tab + hi;          // iv[-i] = 1 / (hi - i)
#pragma unroll 1
        for (int i = 0; i < n4; i += 4) {
            double cv[4];
            if (TABLE) {
#pragma unroll
                for (int u = 0; u < 4; ++u) cv[u] = iv[-(i + u)];
            } else {
                recip4(hi - i, cv);                   // hi - i - 3 >= lo + 1 >= 1
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double r = G * cv[u];
                G *= qi;
                acc0 = fma(r, acc0, r);
                const double rx = r * x;
                acc1 = fma(rx, acc1, rx);
            }
        }
    } else {
#pragma unroll 1
        for (int k = k_top; k >= lo; --k) {
            const double r = G / (double)(k + 1);
            G *= qi;
            acc0 = fma(r, acc0, r);
            const double rx = r * x;
            acc1 = fma(rx, acc1, rx);
        }
    }
    // log((1 + acc1)/(1 + acc0)): the sums are normalised at the window's low
    // end and may exceed the FP32 range, so the ratio stays in double.
    if (rare || !(acc0 < SUM_MAX && acc1 < SUM_MAX)) return delta_ell_rare(mu, d, lmu, lx, win, pc.c, pc.a2);
    return fma((double)lo, (double)lx, log_ratio(1.0 + acc1, 1.0 + acc0) - (double)d);
}

__device__ inline double delta_ell(float mu, float d, const PixConst& pc, const double* inv_tab, int& nterms) {
    return delta_ell_t<true>(mu, d, pc, inv_tab, nterms);
}

// The same without a reciprocal table.  (The scans call their direct evaluations: few
// updates come to them, and inlined they would take the scans' registers.)
__device__ __noinline__ double delta_ell_notab(float mu, float d, const PixConst& pc, int& nterms) {
    return delta_ell_t<false>(mu, d, pc, nullptr, nterms);
}

// Change of the series between displacements y0 = D and y1 = D + d from the
// anchor, as d times the divided difference of the polynomial (Horner on both
// points at once), so it stays proportional to d without cancellation:
// d series_slope(b, D, y1).
__device__ inline float series_slope(float4 b, float D, float y1) {
    float q = b.w;
    float p = fmaf(b.w, D, b.z);
    q = fmaf(q, y1, p);
    p = fmaf(p, D, b.y);
    q = fmaf(q, y1, p);
    p = fmaf(p, D, b.x);
    return fmaf(q, y1, p);
}
__device__ inline float series_delta(float4 b, float D, float d) { return d * series_slope(b, D, D + d); }

// The direct evaluation of the block-series scans, and the series an accepted
// move's pixel takes when it leaves its radius.  Both run over one window, that
// of [mu, mu + d], set up by direct_window: delta_ell_direct sums the two
// Horner recurrences over it, series_after forms the series at mu + d from it
// (the tilted weights W_k x^k are the posterior weights there).
struct DirectWindow {
    double x, qi, G;   // 1 + d / mu, exp(2a), G at the window top
    float lx;          // log x
    int lo, hi, n;     // window [lo, hi), widened to a multiple of four terms
    int terms;         // the window's terms (work measure)
    int kind;          // 0: the recurrence, 1: no value (the caller rejects), 2: sharp read noise
    Window win;        // the window before widening
    float lmu;
};

__device__ inline DirectWindow direct_window(float mu, float d, const PixConst& pc) {
    DirectWindow w;
    w.terms = 0;
    w.kind = 1;
    const float mu1 = mu + d;
    if (!(mu1 > 0.0f) || !(mu > 0.0f)) return w;
    const float t = d * fast_rcp(mu);
    w.lx = log1p_k(t);
    w.lmu = fast_ln(mu);
    w.win = phi_window(w.lmu + fminf(w.lx, 0.0f), w.lmu + fmaxf(w.lx, 0.0f), pc);
    if (!w.win.ok) return w;
    w.terms = w.win.hi - w.win.lo + 1;
    if (pc.a2 > 2.0f * A_RECUR_MAX) {
        w.kind = 2;
        return w;
    }
    w.kind = 0;
    w.lo = w.win.lo;
    w.hi = w.win.hi;
    w.n = (w.hi - w.lo + 3) & ~3;
    w.lo = w.hi - w.n;
    if (w.lo < 0) { w.hi -= w.lo; w.lo = 0; }
    w.x = 1.0 + (double)t;
    w.qi = exp_small(pc.a2);
    w.G = (double)mu * exp_wide_b(-(double)pc.a2 * ((double)(w.hi - 1) + 0.5 - (double)pc.c));
    return w;
}

__device__ inline double direct_sums(float mu, float d, const PixConst& pc, int& nterms) {
    if (d == 0.0f && mu > 0.0f) return 0.0;
    const DirectWindow w = direct_window(mu, d, pc);
    nterms += w.terms;
    if (w.kind == 1) return __builtin_nan("");
    const bool rare = w.kind == 2 || w.win.hi - w.win.lo > LONG_WINDOW;
    // Four Horner steps acc <- (G_u / n_u)(1 + acc) at a time (n_u = hi - i - u,
    // G_u = G qi^u) over their common denominator N = n0 n1 n2 n3:
    //   acc <- G3 [n2 n1 n0 + G2 (n1 n0 + G1 (n0 + G0 (1 + acc)))] / N,
    // one reciprocal per four terms and no per-term one (every quantity is
    // positive, so nothing cancels).  The terms are those of delta_ell_t's
    // recurrence.
    double G = w.G, acc0 = 0.0, acc1 = 0.0;
#pragma unroll 1
    for (int i = 0; i < (rare ? 0 : w.n); i += 4) {
        const double n0 = (double)(w.hi - i), n1 = n0 - 1.0, n2 = n0 - 2.0, n3 = n0 - 3.0;   // n3 >= lo + 1 >= 1
        const double p10 = n1 * n0, p210 = n2 * p10, N = n3 * p210;
        double iN = __builtin_amdgcn_rcp(N);
        iN = fma(iN, fma(-N, iN, 1.0), iN);
        const double g0 = G, g1 = g0 * w.qi, g2 = g1 * w.qi, g3 = g2 * w.qi;
        G = g3 * w.qi;
        double t = fma(g0, acc0, g0) + n0;
        t = fma(g1, t, p10);
        t = fma(g2, t, p210);
        acc0 = (g3 * t) * iN;
        const double x0 = g0 * w.x, x1 = g1 * w.x, x2 = g2 * w.x, x3 = g3 * w.x;
        t = fma(x0, acc1, x0) + n0;
        t = fma(x1, t, p10);
        t = fma(x2, t, p210);
        acc1 = (x3 * t) * iN;
    }
    if (rare || !(acc0 < SUM_MAX && acc1 < SUM_MAX)) return delta_ell_rare(mu, d, w.lmu, w.lx, w.win, pc.c, pc.a2);
    return fma((double)w.lo, (double)w.lx, log_ratio(1.0 + acc1, 1.0 + acc0) - (double)d);
}

__device__ __noinline__ double delta_ell_direct(float mu, float d, const PixConst& pc, int& nterms) {
    return direct_sums(mu, d, pc, nterms);
}

// The two by value, for the nine-phase scan, which comes here more often: its term count
// stays in a register (64 x 64, 20 sweeps: 45.7 ms with the reference's memory, 45.3).
struct DirectValue { double v; int terms; };

__device__ __noinline__ DirectValue direct_value(float mu, float d, PixConst pc) {
    DirectValue r;
    r.terms = 0;
    r.v = direct_sums(mu, d, pc, r.terms);
    return r;
}

__device__ __noinline__ DirectValue notab_value(float mu, float d, PixConst pc) {
    DirectValue r;
    r.terms = 0;
    r.v = delta_ell_t<false>(mu, d, pc, nullptr, r.terms);
    return r;
}

// Lane permutations within rows of 16 (data-parallel primitives, no LDS).
template <int CTRL>
__device__ inline double dpp_d(double v) {
    const int2 u = __builtin_bit_cast(int2, v);
    int2 w;
    w.x = __builtin_amdgcn_update_dpp(0, u.x, CTRL, 0xF, 0xF, false);
    w.y = __builtin_amdgcn_update_dpp(0, u.y, CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, w);
}

__device__ inline double quad_sum(double v) {
    v += dpp_d<0xB1>(v);      // quad_perm [1,0,3,2]
    v += dpp_d<0x4E>(v);      // quad_perm [2,3,0,1]
    return v;
}

// The series at mu + d over the window of [mu, mu + d], by four lanes (p = lane
// mod 4, the same arguments in each, the result in each): lane p takes the
// terms k = lo + p + 4 m.  Its sum over m is one Horner recurrence from the top
// in u = (1 + v)^4 - 1, normalised at its lowest term (as series_at is at lo),
//   A(u) <- R_m (1 + u)(1 + A(u)),  R_m = x^4 G_k G_(k+1) G_(k+2) G_(k+3) /
//   ((k + 1)(k + 2)(k + 3)(k + 4)),
// one reciprocal for the four factors; then u is expanded in v, the lane's
// factor (1 + v)^p W_(lo+p) / W_lo applied and the four lanes added.  A window
// of n terms is n / 4 dependent steps of about 27 issue slots instead of n of 17.
// With d = 0 it is the series at mu from mu's own window.  b2 > 0 and R = 0 where
// no series is formed (a rejected window).
__device__ inline Series series_after(float mu, float d, const PixConst& pc, int p, int& nterms) {
    Series out;
    out.R = 0.0f;
    out.b = no_series();
    const DirectWindow w = direct_window(mu, d, pc);
    if (w.kind == 2) return series_sharp(mu + d, w.win, pc.c, pc.a2);
    if (w.kind != 0) return out;                                    // the same in the four lanes
    nterms += p == 0 ? w.terms : 0;
    // (qi^6 <= exp(480), and the weights' ratios stay in double range with lo as
    // the reference; a factor that underflows belongs to a negligible term, and
    // gx itself does not)
    const double q2 = w.qi * w.qi, q4 = q2 * q2, q6 = q4 * q2;
    // G at the highest index of this lane's first step: hi - 1 for p = 0 (its
    // top term is hi), hi - 5 + p = top - (4 - p) otherwise
    double gx = w.x * (p == 0 ? w.G : w.G * (p == 1 ? q2 * w.qi : (p == 2 ? q2 : w.qi)));
    int m = (w.n >> 2) - (p == 0 ? 1 : 2);
    double k = (double)(w.lo + p + 4 * m);
    double A0 = 0.0, A1 = 0.0, A2 = 0.0, A3 = 0.0, A4 = 0.0;
#pragma unroll 1
    for (; m >= 0; --m) {
        const double t = fma(k, k + 5.0, 4.0), den = t * (t + 2.0); // (k + 1)(k + 4) (k + 2)(k + 3)
        double r = __builtin_amdgcn_rcp(den);
        r = fma(r, fma(-den, r, 1.0), r);
        const double g2 = gx * gx, R = (g2 * q6) * (g2 * r);         // x^4 G_k .. G_(k+3) = (x G_(k+3))^4 qi^6
        gx *= q4;
        k -= 4.0;
        const double T0 = A0 + 1.0;
        A4 = R * (A4 + A3);
        A3 = R * (A3 + A2);
        A2 = R * (A2 + A1);
        A1 = R * (A1 + T0);
        A0 = R * T0;
    }
    // u = 4 v + 6 v^2 + 4 v^3 + v^4
    const double c0 = A0 + 1.0, c1 = 4.0 * A1, c2 = fma(16.0, A2, 6.0 * A1),
                 c3 = fma(64.0, A3, fma(48.0, A2, 4.0 * A1)),
                 c4 = fma(256.0, A4, fma(288.0, A3, fma(68.0, A2, A1)));
    // W_(lo+p) / W_lo: lane 0 ended with x G_(lo+3) qi^4
    const double gl = dpp_d<0x00>(gx);                              // x G_(lo-1)
    const double l1 = (double)(w.lo + 1), l2 = l1 + 1.0, l3 = l1 + 2.0;
    const double l12 = l1 * l2, l123 = l12 * l3;
    double il = __builtin_amdgcn_rcp(p == 3 ? l123 : (p == 2 ? l12 : l1));
    il = fma(il, fma(-(p == 3 ? l123 : (p == 2 ? l12 : l1)), il, 1.0), il);
    const double iq = rcp_nr(w.qi), g1 = gl * iq, g2 = g1 * iq, g3 = g2 * iq;   // x G_lo, x G_(lo+1), x G_(lo+2)
    const double s = p == 0 ? 1.0 : il * (p == 1 ? g1 : (p == 2 ? g1 * g2 : g1 * g2 * g3));
    const double b1 = (double)p, b2 = (double)(p == 3 ? 3 : (p == 2 ? 1 : 0)), b3 = p == 3 ? 1.0 : 0.0;
    const double d0 = c0, d1 = fma(b1, c0, c1), d2 = fma(b2, c0, fma(b1, c1, c2)),
                 d3 = fma(b3, c0, fma(b2, c1, fma(b1, c2, c3))), d4 = fma(b3, c1, fma(b2, c2, fma(b1, c3, c4)));
    const double S0 = quad_sum(s * d0), S1 = quad_sum(s * d1), S2 = quad_sum(s * d2), S3 = quad_sum(s * d3),
                 S4 = quad_sum(s * d4);
    return series_finish(S0, S1, S2, S3, S4, w.lo, mu + d);
}

// A term whose move leaves its series' radius: centre and half-width of an
// interval that holds what the direct evaluation returns.  Anchor m, series
// coefficients b, displacement D (inside the radius), y = D + d, v = y / m.  With p_j =
// sum_i beta_i^j (p_1 = E = (1 + b1) m, p_2 = s2 = -2 b2 m^2, p_3 = 3 b3 m^3, p_4 = -4 b4
// m^4) and T_n the degree-n series of sum_i log(1 + beta_i v), the rest r_n(x) =
// log(1 + x) - x + ... (degree n) satisfies, term by term since 0 < beta < 1,
//   v > 0:  beta^4 |r_3(v)| <= |r_3(beta v)| <= beta^3 |r_3(v)|, r_3 < 0, so
//           T_3 + p_3 r_3(v) <= sum <= T_3 + p_4 r_3(v);
//   v < 0:  T_4 + p_4 r_4(v) <= sum <= T_4 (r_4 < 0, powers of beta fall);
// and, with log(1 + beta v) / beta convex and falling in beta, the chord over
// [0, 1] and Jensen's inequality give for every v > 0, used from v = 1 on,
//   (E^2 / s2) log(1 + s2 v / E) <= sum <= (E - s2) v + s2 log(1 + v).
// At D the series is within TAU / 2.  The direct evaluation and the coefficients round
// too: FP32 logs, a few 1e-7 of E |v|, over 1 - |v| for v < 0 (BND_LOG); and exp(2a) in
// FP32, whose error over a window of n terms is n 1e-7 of the change of the mean count.
// That change is at most (E - s2) |v|, over 1 - |v| for v < 0, as E - s2 is the count's
// variance: next to nothing where read noise is sharp, all of E where it is wide and
// windows are long (BND_EXP, n up to 128 twice and what an earlier window left in the
// coefficients).  log(1 + v) here is off by at most 2e-7 of E; 1e-6 is added.  Over 24 M
// terms of read noise from 0.05 to 100 photons and means from 0.05 to 3000, instructions
// rounded either way, no direct evaluation lay outside (4e-6 of E |v| alone: one in 200 at
// 10 photons).  Not covered: a series formed over the window of a move that took the mean
// to less than 1/100, as its 1 + d / mu is off by more.  Infinite where nothing is
// claimed: no series (b2 > 0), y at the edge of -m, and counts so large that the direct
// window may be refused.
struct TermBound { float c, e; };
constexpr float BND_LOG = 4e-6f, BND_EXP = 6e-5f;
// Of |d|, before the 1 - |v|: m the anchor, b its coefficients, cnt = E / m.
__device__ inline float rounding_of(float m, float4 b, float cnt) {
    return fmaf(BND_EXP, fmaf(2.0f * b.y, m, cnt), BND_LOG * cnt);
}

// sd: series_delta(b, D, y - D).
__device__ inline TermBound series_bound(float m, float4 b, float D, float y, float sd) {
    TermBound t;
    const float v = y * fast_rcp(m), m2 = m * m, v2 = v * v;
    const float E = fmaf(b.x, m, m), s2 = -2.0f * b.y * m2, p3 = 3.0f * b.z * m2 * m, p4 = -4.0f * b.w * m2 * m2;
    const float l = fast_ln(1.0f + v);
    const float r3 = l - v * fmaf(v, fmaf(v, 0.33333333f, -0.5f), 1.0f);
    const float q4 = 0.25f * v2 * v2;
    const float up = v > 0.0f ? p3 * r3 + p4 * q4 : 0.0f, lo = p4 * (r3 + q4);
    t.c = sd + 0.5f * (up + lo);
    t.e = 0.5f * fabsf(up - lo);
    const float ay = fabsf(y), cnt = fabsf(b.x) + 1.0f, den = m - ay;
    float scale = 1.0f;
    if (v < 0.0f) scale = m * fast_rcp(den);
    if (v > 1.0f) {
        const float hi = fmaf(E - s2, v, s2 * l), jn = E * (E * fast_rcp(s2)) * log1p_k(s2 * v * fast_rcp(E));
        // (no count to speak of: the sum lies in [0, E v])
        const float lw = E > 1e-15f && s2 > 1e-15f ? jn : 0.0f;
        t.c = 0.5f * (hi + lw) - y - series_delta(b, 0.0f, D);
        t.e = 0.5f * fabsf(hi - lw);
    }
    t.e = fmaf(scale, fmaf(rounding_of(m, b, cnt), ay + fabsf(D), 1e-6f * cnt * m), t.e + 1.6e-9f);
    if (!(b.y <= 0.0f && (v > 0.0f || den > 0.02f * m) && cnt * (m + ay) < 2.5e5f && t.e < INFINITY)) {
        t.c = 0.0f;
        t.e = INFINITY;
    }
    return t;
}

// Likelihood change of one footprint pixel for the camera the kernel was
// instantiated for (EM: EMCCD reading, one closed-form term; else sCMOS).
template <bool EM>
__device__ inline double delta_pix(float mu, float d, const PixConst& pc, const double* inv_tab, int& nterms) {
    if constexpr (EM) {
        ++nterms;
        return delta_ell_emccd(mu, d, pc);
    } else {
        return delta_ell(mu, d, pc, inv_tab, nterms);
    }
}

__device__ inline Series series_at(float mu, const PixConst& pc, int& nterms) {
    Series out;
    out.b = no_series();
    out.R = 0.0f;
    if (!(mu > 0.0f) || pc.a2 < 0.0f) return out;   // < 0: EMCCD pixel
    const float lmu = fast_ln(mu);
    const Window win = phi_window(lmu, lmu, pc);
    if (!win.ok) return out;
    if (pc.a2 > 2.0f * A_RECUR_MAX) return series_sharp(mu, win, pc.c, pc.a2);
    nterms += win.hi - win.lo + 1;
    // the window widened to a multiple of four terms, as in delta_ell_t
    int lo = win.lo, hi = win.hi;
    const int n4 = (hi - lo + 3) & ~3;
    lo = hi - n4;
    if (lo < 0) { hi -= lo; lo = 0; }
    const double qi = exp_small(pc.a2);
    const int k_top = hi - 1;
    double G = (double)mu * exp_wide_b(-(double)pc.a2 * ((double)k_top + 0.5 - (double)pc.c));
    // A(v) <- r_k (1 + v)(1 + A(v)), coefficients of v^0..v^4, descending so
    // that each update reads the previous step's lower coefficient
    double A0 = 0.0, A1 = 0.0, A2 = 0.0, A3 = 0.0, A4 = 0.0;
#pragma unroll 1
    for (int i = 0; i < n4; i += 4) {
        double cv[4];
        recip4(hi - i, cv);                           // 1/(k+1) for k = k_top - i - u
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double r = G * cv[u];
            G *= qi;
            const double T0 = A0 + 1.0;
            A4 = r * (A4 + A3);
            A3 = r * (A3 + A2);
            A2 = r * (A2 + A1);
            A1 = r * (A1 + T0);
            A0 = r * T0;
        }
    }
    return series_finish(1.0 + A0, A1, A2, A3, A4, lo, mu);
}

}  // namespace bdc
