// bdc_bounds.h -- the interval of one footprint term of the bounded block pass: the
// change of a pixel's log-likelihood (either camera) from the local series of an anchor
// that may lie behind the present mean.
#pragma once

#include "bdc_device.h"

namespace bdc {

constexpr float BND_R = 6.0f;                    // reach of a series that bounds only, in radii

// Series of log f of an EMCCD pixel at mean mu, and what B f is there beside A: its share
// w = B f / (A + B f), or, from lam = log(B f / A) = EM_LAM on, where 1 - w leaves FP32,
// lam itself (so a value below 1 is a share).
struct EmSeries { Series s; float w; };
constexpr float EM_LAM = 16.0f;

__device__ __noinline__ EmSeries emccd_series(float muf, float cf, float lA, float lB) {
    EmSeries o;
    o.s.R = 0.0f;
    o.s.b = no_series();
    o.w = INFINITY;
    if (!(muf > 0.0f)) return o;
    if (!(cf > 0.0f)) {                                             // no photon amplified: exactly -mu
        o.s.b = make_float4(-1.0f, 0.0f, 0.0f, 0.0f);
        o.s.R = muf;
        return o;
    }
    const double mu = (double)muf, c = (double)cf, q = mu * c, z = 2.0 * sqrt(q);
    double lf;
    if (z < 16.0) {
        // t_k = q^k / (k! (k + 1)!):  sum t_k = 2 I_1 / z, sum (k + 1) t_k = I_0;
        // mu f' / f = their ratio E, mu^2 f'' = q f
        double t = 1.0, s0 = 1.0, s1 = 1.0;
#pragma unroll 4
        for (int k = 1; k < 64; ++k) {
            t *= q * rcp_nr((double)(k * (k + 1)));
            s1 += t;
            s0 = fma((double)(k + 1), t, s0);
            if (t < 1e-13 * s1) break;
        }
        const double E = s0 * rcp_nr2(s1);
        lf = (double)fast_ln((float)(mu * s1));
        o.s = series_finish(1.0, E, 0.5 * q, q * (E - 1.0) * (1.0 / 6.0), q * (q - 2.0 * E + 2.0) * (1.0 / 24.0), 0,
                            muf);
    } else {
        // log f = log(mu / c) / 2 + z - log(2 pi z) / 2 + l(z), z ~ (1 + v)^(1/2) and
        // l = -3/8 / z - 3/16 / z^2 - 21/128 / z^3 - 0.2109 / z^4 (Hankel's series)
        const float zf = (float)z, i1 = fast_rcp(zf), l1 = -0.375f * i1, l2 = -0.1875f * i1 * i1,
                    l3 = -0.1640625f * i1 * i1 * i1, l4 = -0.2109f * i1 * i1 * i1 * i1;
        const float g1 = 0.5f * zf + 0.25f - 0.5f * l1 - l2 - 1.5f * l3 - 2.0f * l4;
        const float g2 = -0.125f * zf - 0.125f + 0.375f * l1 + l2 + 1.875f * l3 + 3.0f * l4;
        const float g3 = 0.0625f * zf + 0.083333333f - 0.3125f * l1 - l2 - 2.1875f * l3 - 4.0f * l4;
        const float g4 = -0.0390625f * zf - 0.0625f + 0.2734375f * l1 + l2 + 2.4609375f * l3 + 5.0f * l4;
        lf = (double)(0.5f * (fast_ln(muf * fast_rcp(cf)) - fast_ln(6.2831853f * zf)) + (l1 + l2 + l3 + l4)) + z;
        o.s = series_of_log(g1, g2, g3, g4, muf);
    }
    const float lam = (float)((double)lB + lf - (double)lA);         // log(B f / A)
    o.w = lam < EM_LAM ? fast_rcp(1.0f + __builtin_amdgcn_exp2f(-1.44269504f * lam)) : lam;
    if (!(o.s.b.y <= 0.0f)) {
        o.s.b = no_series();
        o.s.R = 0.0f;
    }
    return o;
}

// log(1 + w (e^g - 1)), 0 <= w <= 1, and the argument of the logarithm.
__device__ inline float em_mix(float w, float g, float& arg) {
    arg = fmaf(w, __builtin_amdgcn_exp2f(g * 1.44269504f) - 1.0f, 1.0f);
    return fast_ln(arg);
}

// Centre and half-width of the term's interval: anchor A.x, reach A.y and coefficients of
// the pixel's series (A.z, A.w, B), present mean mu, change d; out: mu + d lies beyond the
// reach.  Half-width infinite (centre 0) where nothing is claimed.
//
// EMCCD: with D = mu - A.x and g the change of log f from the anchor, the term is the
// change of log(A + B f e^g).  While the anchor's share w is told, that is
// log(1 + w (e^g - 1)) at both points.  Beyond EM_LAM it is g + log(1 + e^-(lam + g)); the
// second term is left out and its bound e^-(lam + g), at the lower of the two points
// and with g less its own half-width, added to the half-width (the factor e covers
// the rounding of lam and g): at a drifted anchor, or down from a bright pixel, it need
// not be small.
template <bool EM>
__device__ inline TermBound bounded_term(float4 A, float2 Bv, float share, float mu, float d, bool out) {
    TermBound t;
    const float4 b = make_float4(A.z, A.w, Bv.x, Bv.y);
    const float D = mu - A.x, y = D + d, cnt = fabsf(b.x) + 1.0f;
    const float ym = out ? fabsf(D) : fmaxf(fabsf(y), fabsf(D)), y2 = ym * ym;
    const float trunc = fabsf(b.w) * (y2 * y2) * (3.2f * ym * fast_rcp(A.x));
    t.c = d * series_slope(b, D, y);
    t.e = rounding_of(A.x, b, cnt) * fabsf(d);
    if (out) t = series_bound(A.x, b, D, y, t.c);
    if (EM) {
        const float gD = fmaf(D, series_slope(b, 0.0f, D), D), gy = gD + t.c + d;
        if (share < 1.0f) {
            float ay, aD;
            const float my = em_mix(share, gy, ay), mD = em_mix(share, gD, aD);
            t.c = my - mD - d;
            // rounding of the share, exponentials, arguments and logarithms
            t.e += fmaf(5e-7f, fabsf(gy) + fabsf(gD), 5e-6f) + 5e-7f * fast_rcp(fminf(ay, aD)) + 4e-6f * cnt * fabsf(D);
            if (!(gy < 60.0f && ay > 0.0f && aD > 0.0f)) t.e = INFINITY;
        } else {
            t.e += __builtin_amdgcn_exp2f(1.44269504f * (1.0f + t.e - share - fminf(gy, gD)));
        }
    }
    t.e += trunc;
    if (!(t.e < INFINITY)) {
        t.c = 0.0f;
        t.e = INFINITY;
    }
    return t;
}

}  // namespace bdc
