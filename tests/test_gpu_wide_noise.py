"""Sweeps of cameras with wide read noise decide as the direct evaluations do."""

import numpy as np
import pytest

from paper_2411_00991_amd import synth
from test_gpu_decisions import advance_by_groups, bdc, frame, lattice_frame, twins  # noqa: F401

pytestmark = pytest.mark.gpu


# (schedule, object sub-lattice, psf, h, w, level, read noise in ADU of the left half, G = 2): means up to some
# hundred photons, noise of 3.5 to 40 photons, so that windows of hundreds of terms are met beside short ones
@pytest.mark.parametrize("case", [("SERIES", 1, 25, 60, 55, 10.0, 7.0), ("SERIES", 1, 31, 64, 70, 20.0, 24.0),
                                  ("SERIES9", 1, 11, 40, 44, 10.0, 30.0), ("SERIES9", 1, 15, 45, 40, 30.0, 80.0),
                                  ("BLOCK", 2, 15, 30, 33, 10.0, 24.0)],
                         ids=lambda c: "%s-k%d-%d-%gx%g" % (c[0], c[1], c[2], c[5], c[6]))
def test_sweeps_reach_the_state_of_direct_decisions(bdc, case):  # noqa: F811
    sched, k, s, h, w, level, noise = case
    psf = synth.gaussian_psf(max(0.5, (s - 1) / 8.0), s)
    if k == 1:
        img, cam = frame(h, w, psf, 40 + s, level, noise)
    else:
        img, cam = lattice_frame(h, w, k, psf, 40 + s, 0, level, noise)
    sid = {"SERIES": bdc.BDC_SCHED_BLOCK_SERIES, "SERIES9": bdc.BDC_SCHED_BLOCK9_SERIES, "BLOCK": bdc.BDC_SCHED_BLOCK}[sched]
    A, B = twins(bdc, img, cam, psf, sid, 0, 2, 5 + s, 4, object_sub=k)
    A.sweep(6)
    advance_by_groups(B, 6)
    ra, la, _ = A.rho()
    rb, lb, _ = B.rho()
    assert np.array_equal(ra, rb) and np.array_equal(la, lb)


# EMCCD: zero-photon normal of 8 to 60 photons' width, so that it and the amplified photons take turns in dominating
@pytest.mark.parametrize("s,level,noise", [(11, 5.0, 16.0), (15, 40.0, 60.0), (21, 20.0, 120.0)])
def test_emccd_sweeps_reach_the_state_of_direct_decisions(bdc, s, level, noise):  # noqa: F811
    psf = synth.gaussian_psf((s - 1) / 8.0, s)
    img, cam = lattice_frame(45, 50, 1, psf, 60 + s, 1, level, noise)
    A, B = twins(bdc, img, cam, psf, bdc.BDC_SCHED_BLOCK, 0, 2, 5 + s, 4, camera=1)
    A.sweep(6)
    advance_by_groups(B, 6)
    ra, la, _ = A.rho()
    rb, lb, _ = B.rho()
    assert np.array_equal(ra, rb) and np.array_equal(la, lb)
