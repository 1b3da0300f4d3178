"""The likelihood terms of the device code, compiled for the host.

The arithmetic of bdc_device.h runs here with the gfx950 instructions it calls replaced by exact ones
and by ones that err by a unit in the last place, over ranges that no frame of the GPU tests covers:
read noise from a twentieth of a photon to a hundred, moves by large factors.
"""

import ctypes
import os
import subprocess

import numpy as np
import pytest
from scipy.special import gammaln

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")


@pytest.fixture(scope="module", params=["exact", "ulp"])
def terms(request, tmp_path_factory):
    out = str(tmp_path_factory.mktemp("terms") / "libterms.so")
    subprocess.check_call(["g++", "-O2", "-std=c++20", "-w", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "paper_2411_00991_amd", "csrc"), "-I", HOST] +
                          (["-DULP"] if request.param == "ulp" else []) +
                          [os.path.join(HOST, "terms.cpp"), "-o", out])
    return ctypes.CDLL(out)


def call(fn, n, ins, outs):
    """fn(n, inputs as float32, outputs of the given dtypes)"""
    ins = [np.ascontiguousarray(v, np.float32) for v in ins]
    res = [np.empty(n, t) for t in outs]
    fn(ctypes.c_int(n), *[ctypes.c_void_p(v.ctypes.data) for v in ins + res])
    return res


def exact_delta(c, a, mu, d):
    """log-likelihood change of the sCMOS pixel in float64, over every count that matters"""
    k = np.arange(0.0, 2.0 * max(c, mu, mu + d) + 3000.0)
    lw = -a * (k - c) ** 2 - gammaln(k + 1.0)
    ell = lambda m: np.logaddexp.reduce(lw + k * np.log(m)) - m
    return ell(mu + d) - ell(mu)


def wide_noise_cases(n):
    """Pixels of wide read noise (10 to 100 photons), moves up to factors of e^3 either way."""
    rng = np.random.default_rng(3)
    sg = np.exp(rng.uniform(np.log(10.0), np.log(100.0), n))
    m = np.exp(rng.uniform(np.log(0.5), np.log(3000.0), n))
    c = np.float32(rng.poisson(m) + sg * rng.standard_normal(n))
    mu = np.float32(m * np.exp(rng.normal(0.0, 0.7, n)))
    d = np.float32(mu * np.expm1(np.clip(rng.normal(0.0, 1.2, n), -3.0, 3.0)))
    fixed = np.array([(482.0, 2 * 0.00317, 480.0, -469.0), (1008.48, 2 * 0.001392, 652.569, -607.855),
                      (482.0, 2 * 0.00317, 11.0, 469.0)], np.float32)
    return [np.concatenate([v, fixed[:, k]]) for k, v in enumerate([c, np.float32(1.0 / sg ** 2), mu, d])]


def test_long_windows_of_wide_read_noise(terms):
    """Windows of more than 128 terms: no sum overflows, no error of exp(2a) accumulates.  The
    window leaves out weights of e^-20 (2e-9) of a sum each side, the rest is double precision."""
    c, a2, mu, d = wide_noise_cases(400)
    a2, out, out2, longer = call(terms.direct, len(c), [c, a2, mu, d], [np.float32, np.float64, np.float64, np.int32])
    assert longer.sum() > 200 and longer[-3:].all()
    for i in np.flatnonzero(longer):
        ref = exact_delta(float(c[i]), 0.5 * float(a2[i]), float(mu[i]), float(d[i]))
        tol = 1e-8 + 1e-11 * abs(ref) + 1e-11 * abs(d[i])
        assert abs(out[i] - ref) <= tol, (c[i], a2[i], mu[i], d[i], out[i], ref)
        assert abs(out2[i] - ref) <= tol, (c[i], a2[i], mu[i], d[i], out2[i], ref)


def test_sums_that_overflow_in_short_windows(terms):
    """A mode far above the window's end in fewer than 129 terms, as after a jump by a factor of 1e5."""
    rng = np.random.default_rng(4)
    n = 300
    a2 = np.float32(np.exp(rng.uniform(np.log(0.12), np.log(0.3), n)))
    c = np.float32(rng.uniform(300.0, 900.0, n))
    hi = np.float32(c * np.exp(rng.normal(0.0, 0.3, n)))
    lo = np.float32(hi * np.exp(-rng.uniform(8.0, 17.0, n)))
    up = rng.random(n) < 0.5
    mu = np.where(up, lo, hi)
    d = np.float32(np.where(up, hi - lo, lo - hi))
    a2, out, out2, longer = call(terms.direct, n, [c, a2, mu, d], [np.float32, np.float64, np.float64, np.int32])
    # (a mean that 1 + d / mu in FP32 does not tell from zero has no value)
    short = (longer == 0) & (mu + d > np.float32(1e-6) * mu)
    assert short.sum() > 50
    for i in np.flatnonzero(short):
        ref = exact_delta(float(c[i]), 0.5 * float(a2[i]), float(mu[i]), float(d[i]))
        # FP32: log x (2^-23 of it times the lowest count), x = 1 + d / mu near 0 (2^-23 / x of the count)
        x = min(1.0, (float(mu[i]) + float(d[i])) / float(mu[i]))
        tol = 1e-4 + (c[i] + 200.0) * (3e-7 / max(x, 1e-9) + 1e-5)
        assert abs(out[i] - ref) <= tol, (c[i], a2[i], mu[i], d[i], out[i], ref)
        assert abs(out2[i] - ref) <= tol, (c[i], a2[i], mu[i], d[i], out2[i], ref)


@pytest.mark.parametrize("noise", [(0.05, 0.5), (0.5, 2.0), (2.0, 5.0), (5.0, 10.0), (10.0, 20.0), (20.0, 100.0)],
                         ids=lambda v: "%gto%g" % v)
def test_intervals_hold_the_direct_evaluation(terms, noise):
    """What a scan decides from: the direct evaluation lies within 1.02 half-widths and 1e-7 of the
    centre, at any read noise, anchored at a mean of its own or after a move by up to a factor of
    e^6 up and 1/100 down, for moves by factors of e^-4 to e^6."""
    rng = np.random.default_rng(int(noise[0] * 100))
    n = 120000
    sg = np.exp(rng.uniform(np.log(noise[0]), np.log(noise[1]), n))
    true = np.exp(rng.uniform(np.log(0.05), np.log(3000.0), n))
    c = np.float32(rng.poisson(true) + sg * rng.standard_normal(n))
    m = np.float32(true * np.exp(rng.normal(0.0, 0.7, n)))
    last = np.clip(rng.normal(0.0, 1.0, n) * np.where(rng.random(n) < 0.5, 0.3, 2.0), -6.0, 4.6)
    m0 = np.where(rng.random(n) < 0.4, np.float32(0.0), np.float32(m * np.exp(last)))
    dm = np.float32(m - m0)
    shift = np.where(rng.random(n) < 0.3, 0.0, rng.uniform(-1.0, 1.0, n))
    step = np.expm1(np.clip(rng.normal(0.0, 1.0, n) * np.where(rng.random(n) < 0.6, 0.5, 2.0), -4.0, 6.0))
    centre, half, value, radius = call(terms.bounds, n, [c, np.float32(1.0 / sg ** 2), m0, dm, shift, step], [np.float64] * 4)
    tell = (radius > 0.0) & np.isfinite(half) & np.isfinite(centre)
    assert tell.mean() > 0.3
    excess = np.abs(value - centre) - (1.02 * half + 1e-7)
    assert np.isfinite(value[tell]).all()
    assert excess[tell].max() <= 0.0, (excess[tell].max(), np.flatnonzero(tell)[excess[tell].argmax()])


@pytest.mark.parametrize("noise", [(0.3, 3.0), (3.0, 20.0), (20.0, 100.0)], ids=lambda v: "%gto%g" % v)
def test_emccd_intervals_hold_the_direct_evaluation(terms, noise):
    """The reading is a mixture of the zero-photon normal (A) and the amplified photons (B f): an
    interval of the bounded pass holds its direct evaluation whichever of the two dominates at the
    anchor, at the present mean (anywhere in the series' reach) and at the proposed one.  The pass
    adds 1.3e-6 of the centre and 1e-7 a term, and decides at 1.02 half-widths and 1e-7."""
    rng = np.random.default_rng(int(noise[0] * 100))
    n = 150000
    sg = np.exp(rng.uniform(np.log(noise[0]), np.log(noise[1]), n))          # read noise over gain, photons
    gain = 20.0
    true = np.exp(rng.uniform(np.log(0.02), np.log(3000.0), n))
    phi = rng.poisson(true)
    c = np.where(phi > 0, rng.gamma(np.maximum(phi, 1), 1.0), sg * rng.standard_normal(n))
    m = true * np.exp(rng.normal(0.0, 0.8, n))
    shift = np.where(rng.random(n) < 0.2, 0.0, rng.uniform(-1.0, 1.0, n))
    step = np.expm1(np.clip(rng.normal(0.0, 1.0, n) * np.where(rng.random(n) < 0.6, 0.3, 2.0), -3.8, 6.0))
    # a mean drifted by the whole reach to where A dominates; A only just out of FP32's sight
    sg[:2], c[:2], m[:2], shift[:2], step[:2] = [87.9, 36.0], [1910.92, 89.7], [375.136, 29.5], [-0.997, 0.0], [0.0918, -0.2045]
    c = np.float32(c)
    s = sg * gain
    lA = -0.5 * np.log(2.0 * np.pi * s ** 2) - (c.astype(np.float64) * gain) ** 2 / (2.0 * s ** 2)
    lB = np.where(c > 0, -c.astype(np.float64) - np.log(gain), -np.inf)
    centre, half, value = call(terms.emccd, n, [c, lA, lB, m, shift, step], [np.float64] * 3)
    tell = np.isfinite(half)
    assert tell.mean() > 0.7
    excess = np.abs(value - centre) - (1.02 * (half + 1.3e-6 * np.abs(centre) + 1e-7) + 1e-7)
    assert np.isfinite(value[tell]).all()
    assert excess[tell].max() <= 0.0, (excess[tell].max(), np.flatnonzero(tell)[excess[tell].argmax()])
