"""Sweeps decide most moves from certified bounds instead of direct evaluations.

The parity hook always forms Delta itself (every term outside its series'
radius evaluated directly), so a chain advanced by it group by group is the
reference: a chain advanced by plain sweeps must reach the same state bit for
bit, steps included, in every scan that decides by bounds.
"""

import numpy as np
import pytest

from paper_2411_00991_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bdc():
    import torch
    torch.cuda.set_device(0)
    import paper_2411_00991_amd as m
    return m


def f32(a):
    return np.asarray(a, np.float32)


def frame(h, w, psf, seed, level=1.0, sharp=0.0):
    """Beads on a gradient background; level scales the light, sharp (a read noise) puts such pixels in the left half."""
    rng = np.random.default_rng(seed)
    obj = np.broadcast_to(np.linspace(1.0, 8.0, w)[None, :], (h, w)).copy()
    synth.add_beads(obj, rng, max(4, h * w // 150))
    cam = synth.scmos_maps(rng, h, w)
    if sharp:
        cam.sigma[:, :w // 2] = sharp
    return synth.simulate_frame(obj * level, psf, cam, rng), cam


def twins(bdc, img, cam, psf, schedule, block, chains, seed, burn, **kw):
    out = []
    for _ in range(2):
        h, w = img.shape
        S = bdc.Sampler(f32(psf), *[f32(a) for a in cam.maps(h, w)], height=h, width=w, n_chains=chains, seed=seed,
                        burn_in=burn, schedule=schedule, block_size=block, log_step0=-0.3, **kw)
        S.init(f32(img))
        out.append(S)
    return out


def advance_by_groups(S, sweeps):
    n = S.schedule_info()[0]
    for _ in range(sweeps):
        S.run_groups(0, n)
        rho, ls, t = S.rho()
        S.set_rho(rho, ls, t + 1)


SERIES_CASES = [
    # (schedule, block, psf, h, w, level, read noise of the left half where not 0)
    ("SERIES", 0, ("airy", 31), 70, 97, 1.0, 0.0),
    ("SERIES", 31, ("airy", 31), 64, 64, 20.0, 0.0),
    ("SERIES", 0, ("airy", 31), 66, 62, 0.05, 0.0),
    ("SERIES", 0, ("gauss", 21), 61, 50, 1.0, 0.15),
    ("SERIES", 0, ("gauss", 3), 23, 31, 3.0, 0.0),
    ("SERIES", 0, ("airy", 27), 60, 57, 60.0, 0.24),         # 2a just below the recurrence's limit
    ("SERIES9", 0, ("gauss", 11), 40, 36, 40.0, 0.24),
    ("SERIES9", 0, ("gauss", 11), 36, 40, 0.2, 0.26),
    ("SERIES9", 0, ("gauss", 11), 64, 64, 1.0, 0.0),
    ("SERIES9", 11, ("gauss", 11), 45, 71, 30.0, 0.0),
    ("SERIES9", 5, ("gauss", 11), 40, 40, 0.03, 0.0),
    ("SERIES9", 0, ("gauss", 9), 37, 50, 1.0, 0.15),
    ("SERIES9", 0, ("airy", 21), 80, 60, 1.0, 0.0),
    ("SERIES9", 0, ("airy", 31), 64, 70, 1.0, 0.15),
    ("SERIES9", 0, ("gauss", 3), 19, 26, 2.0, 0.0),
    ("SERIES9", 0, ("gauss", 13), 40, 45, 1.0, 0.0),         # either side of 4, 6 and 7 entries per lane
    ("SERIES9", 0, ("gauss", 17), 50, 41, 5.0, 0.0),
    ("SERIES9", 0, ("airy", 19), 57, 60, 1.0, 0.0),
    ("SERIES9", 0, ("gauss", 23), 60, 52, 1.0, 0.0),
]


@pytest.mark.parametrize("case", SERIES_CASES, ids=lambda c: "%s-B%d-%s%d-%gx%g" % (c[0], c[1], *c[2], c[5], c[6]))
def test_sweeps_reach_the_state_of_direct_decisions(bdc, case):
    sched, block, (kind, s), h, w, level, sharp = case
    psf = synth.gaussian_psf(max(0.5, (s - 1) / 8.0), s) if kind == "gauss" else synth.airy_psf_matched(s / 10.0, s)
    img, cam = frame(h, w, psf, 17 + s + h, level, sharp)
    sid = {"SERIES": bdc.BDC_SCHED_BLOCK_SERIES, "SERIES9": bdc.BDC_SCHED_BLOCK9_SERIES}[sched]
    A, B = twins(bdc, img, cam, psf, sid, block, 2, 5 + s, 4)
    A.profile_read()
    A.sweep(6)
    work = A.profile_read()[2]
    print(case, "direct evaluations %d of %d" % (work[2], work[1]), flush=True)
    advance_by_groups(B, 6)
    ra, la, ta = A.rho()
    rb, lb, tb = B.rho()
    assert ta == tb == 6
    assert np.array_equal(ra, rb) and np.array_equal(la, lb)


def lattice_frame(h, w, k, psf, seed, emccd, level, sharp):
    """The same object on a k times finer lattice, read by either camera."""
    from scipy import signal
    rng = np.random.default_rng(seed)
    obj = np.broadcast_to(np.linspace(1.0, 8.0, w * k)[None, :], (h * k, w * k)) / k ** 2
    obj = obj.copy()
    synth.add_beads(obj, rng, max(4, h * w // 150), scale=50.0 / k ** 2)
    mu = np.clip(signal.fftconvolve(obj * level, psf, mode="same"), 1e-6, None)
    phi = rng.poisson(mu.reshape(h, k, w, k).sum(axis=(1, 3)))
    cam = synth.scmos_maps(rng, h, w)
    if sharp:
        cam.sigma[:, :w // 2] = sharp
    g, o, sg = cam.maps(h, w)
    if emccd:
        img = o + g * np.where(phi > 0, rng.gamma(np.maximum(phi, 1), 1.0), 0.0)
        return img + np.where(phi == 0, sg * rng.standard_normal((h, w)), 0.0), cam
    return g * phi + o + sg * rng.standard_normal((h, w)), cam


# One cell per block and colour, without a series scan of its own: the EMCCD reading, the chunk prior, a finer lattice.
# Footprints on both sides of every launch size (F = 256, 512, 1024, 1536 terms; pixel side 33 at k = 2 and PSF 63),
# blocks of s - 1, and one region (EMCCD, side 37) beyond the LDS, which takes the direct pass.
BOUNDED_CASES = [
    # (EMCCD, chunk prior, k, psf, block, h, w, level, read noise of the left half where not 0)
    (1, 0, 1, ("gauss", 3), 3, 20, 31, 1.0, 0.0),
    (1, 0, 1, ("gauss", 11), 0, 40, 37, 0.05, 0.0),
    (1, 0, 1, ("gauss", 15), 14, 45, 50, 20.0, 0.0),
    (1, 0, 1, ("airy", 17), 0, 40, 61, 1.0, 0.1),
    (1, 0, 1, ("airy", 23), 22, 50, 60, 1.0, 0.0),
    (1, 0, 1, ("airy", 33), 0, 70, 67, 5.0, 0.0),
    (1, 0, 1, ("gauss", 37), 0, 75, 80, 1.0, 0.0),
    (0, 1, 1, ("gauss", 3), 2, 19, 22, 1.0, 0.0),
    (0, 1, 1, ("gauss", 11), 0, 37, 45, 0.1, 0.15),
    (0, 1, 1, ("gauss", 15), 14, 44, 43, 30.0, 0.0),
    (0, 1, 1, ("airy", 21), 20, 50, 61, 1.0, 0.0),
    (0, 1, 1, ("airy", 31), 0, 63, 80, 1.0, 0.0),
    (1, 1, 1, ("gauss", 15), 0, 40, 47, 1.0, 0.0),
    (1, 1, 1, ("airy", 31), 30, 64, 70, 2.0, 0.0),
    (0, 0, 2, ("gauss", 15), 0, 30, 33, 1.0, 0.0),
    (0, 0, 2, ("airy", 31), 0, 40, 45, 10.0, 0.15),
    (0, 0, 2, ("airy", 63), 0, 70, 68, 1.0, 0.0),
    (0, 0, 3, ("gauss", 31), 0, 30, 29, 0.1, 0.0),
    (1, 0, 2, ("airy", 41), 0, 50, 47, 1.0, 0.0),
    (1, 0, 2, ("airy", 63), 0, 67, 66, 1.0, 0.0),
]


@pytest.mark.parametrize("case", BOUNDED_CASES,
                         ids=lambda c: "em%d-dir%d-k%d-%s%d-B%d-%gx%g" % (*c[:3], *c[3], c[4], *c[7:]))
def test_bounded_block_sweeps_reach_the_state_of_direct_decisions(bdc, case):
    em, chunk, k, (kind, s), block, h, w, level, sharp = case
    psf = synth.gaussian_psf(max(0.5, (s - 1) / 8.0), s) if kind == "gauss" else synth.airy_psf_matched(s / 10.0, s)
    img, cam = lattice_frame(h, w, k, psf, 11 + s + h, em, level, sharp)
    A, B = twins(bdc, img, cam, psf, bdc.BDC_SCHED_BLOCK, block, 2, 5 + s, 3, camera=em, object_sub=k,
                 prior_kind=bdc.BDC_PRIOR_DIRICHLET if chunk else bdc.BDC_PRIOR_FLAT)
    A.profile_read()
    A.sweep(4)
    work = A.profile_read()[2]
    print(case, "direct evaluations %d of %d" % (work[2], work[1]), flush=True)
    advance_by_groups(B, 4)
    ra, la, ta = A.rho()
    rb, lb, tb = B.rho()
    assert ta == tb == 4
    assert np.array_equal(ra, rb) and np.array_equal(la, lb)


def test_colour_ranges_of_the_bounded_block_pass(bdc):
    """Group ranges cut anywhere (mid-row, mid-phase) visit every cell once between them."""
    psf = synth.gaussian_psf(1.5, 11)
    img, cam = lattice_frame(29, 34, 2, psf, 3, 1, 1.0, 0.0)
    A, B = twins(bdc, img, cam, psf, bdc.BDC_SCHED_BLOCK, 0, 2, 9, 3, camera=1, object_sub=2)
    n = A.schedule_info()[0]
    cuts = [0, 7, n // 3, n // 3 + 1, n // 2 + 5, n]
    visits = np.zeros((2, 58, 68), int)
    for a, b in zip(cuts[:-1], cuts[1:]):
        visits += B.run_groups(a, b)[1] != 255
    assert np.all(visits == 1)
    assert np.all(A.run_groups(0, n)[1] != 255)
