// The likelihood terms of bdc_device.h and bdc_bounds.h on the host, for test_term_bounds.py.
#include "builtins.h"

#include "bdc_bounds.h"

using namespace bdc;

// Per-pixel constants as the frame set-up stores them and the kernels load them.
static PixConst make_pc(double c, double a) {
    PixConst p;
    const double ks = c > 0.0 ? c : 0.0;
    p.c = (float)c;
    p.a2 = record_a2((float)(2.0 * a));
    p.ks = fmaxf(p.c, 0.0f);
    p.L0 = (float)(2.0 * a * (c - ks) - std::log(ks + 1.0));
    p.iB = (float)(1.0 / (2.0 * a + 1.0 / (ks + 1.0)));
    p.inv2a = 1.0f / p.a2;
    p.h0 = std::sqrt(2.0f * TAIL_T * p.inv2a);
    return p;
}

extern "C" {

// The two direct evaluations; a2: in, and as the record holds it; longer: whether the
// window counts as long.
void direct(int n, const float* c, const float* a2, const float* mu, const float* d, float* held, double* out, double* out2,
            int* longer) {
    for (int i = 0; i < n; ++i) {
        const PixConst pc = make_pc(c[i], 0.5 * (double)a2[i]);
        int terms = 0;
        held[i] = pc.a2;
        out[i] = delta_ell_direct(mu[i], d[i], pc, terms);
        out2[i] = delta_ell_notab(mu[i], d[i], pc, terms);
        const Window w = direct_window(mu[i], d[i], pc).win;
        longer[i] = w.hi - w.lo > LONG_WINDOW;
    }
}

// Interval and direct evaluation of moves mu -> mu + d, mu = m + shift R, of a pixel whose
// series was formed at m = m0 + dm: over the window of that move, or (m0 = 0) over its
// own.  radius: R, -1 where no series was formed.
void bounds(int n, const float* c, const float* a2, const float* m0, const float* dm, const float* shift, const float* step,
            double* centre, double* half, double* value, double* radius) {
    for (int i = 0; i < n; ++i) {
        const PixConst pc = make_pc(c[i], 0.5 * (double)a2[i]);
        int terms = 0;
        const float m = m0[i] + dm[i];
        Series s;
        if (m0[i] > 0.0f) {
            quad.run([&](int lane) {
                Series one = series_after(m0[i], dm[i], pc, lane, terms);
                if (lane == 0) s = one;
            }, 4);
        } else {
            s = series_at(m, pc, terms);
        }
        const float mu = m + shift[i] * s.R, d = mu * step[i], D = mu - m, y = D + d;
        const TermBound t = series_bound(m, s.b, D, y, series_delta(s.b, D, d));
        centre[i] = t.c;
        half[i] = t.e;
        value[i] = delta_ell_direct(mu, d, pc, terms);
        radius[i] = s.b.y <= 0.0f ? (fabsf(y) <= s.R ? 0.0 : (double)s.R) : -1.0;
    }
}

// EMCCD: interval of the bounded pass and direct evaluation of moves mu -> mu + d, mu = m +
// shift times the reach of the series at m, with the record's log A and -c - log G.
void emccd(int n, const float* c, const float* lA, const float* lB, const float* m, const float* shift, const float* step,
           double* centre, double* half, double* value) {
    for (int i = 0; i < n; ++i) {
        const EmSeries es = emccd_series(m[i], c[i], lA[i], lB[i]);
        const float reach = m[i] * (fabsf(es.s.b.x) + 1.0f) < 1e5f ? fminf(BND_R * es.s.R, 0.5f * m[i]) : 0.0f;
        const float mu = m[i] + shift[i] * reach, d = mu * step[i];
        PixConst pc;
        pc.c = c[i];
        pc.a2 = -1.0f;
        pc.L0 = lA[i];
        pc.iB = lB[i];
        const bool out = !(fabsf((mu - m[i]) + d) <= reach);
        const TermBound t = bounded_term<true>(make_float4(m[i], reach, es.s.b.x, es.s.b.y), make_float2(es.s.b.z, es.s.b.w),
                                               es.w, mu, d, out);
        centre[i] = t.c;
        half[i] = t.e;
        value[i] = delta_ell_emccd(mu, d, pc);
    }
}

}  // extern "C"
