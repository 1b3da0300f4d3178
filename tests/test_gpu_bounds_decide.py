"""The scans that decide from bounds do so: in the cases that compare them with direct decisions most
footprint terms are never evaluated directly, and the one region beyond the LDS takes the all-direct pass."""

import pytest

from paper_2411_00991_amd import synth
from test_gpu_decisions import BOUNDED_CASES, SERIES_CASES, bdc, frame, lattice_frame, twins  # noqa: F401

pytestmark = pytest.mark.gpu


def work_of(S, sweeps):
    S.profile_read()
    S.sweep(sweeps)
    terms, evals, direct, anchors = S.profile_read()[2][:4]
    return evals, direct, anchors


@pytest.mark.parametrize("case", SERIES_CASES, ids=lambda c: "%s-B%d-%s%d-%gx%g" % (c[0], c[1], *c[2], c[5], c[6]))
def test_series_scans_decide_from_bounds(bdc, case):  # noqa: F811
    sched, block, (kind, s), h, w, level, sharp = case
    psf = synth.gaussian_psf(max(0.5, (s - 1) / 8.0), s) if kind == "gauss" else synth.airy_psf_matched(s / 10.0, s)
    img, cam = frame(h, w, psf, 17 + s + h, level, sharp)
    sid = {"SERIES": bdc.BDC_SCHED_BLOCK_SERIES, "SERIES9": bdc.BDC_SCHED_BLOCK9_SERIES}[sched]
    S = twins(bdc, img, cam, psf, sid, block, 2, 5 + s, 4)[0]
    evals, direct, anchors = work_of(S, 6)
    assert anchors > 0
    # the nine-phase scan's queue holds 64 terms at side 31 and gives no bound beyond, so that updates over
    # hundreds of sharp pixels (none of which has a radius) stay with their direct evaluations
    if not (sched == "SERIES9" and s > 21 and sharp):
        assert 0 <= direct < 0.5 * evals


@pytest.mark.parametrize("case", BOUNDED_CASES,
                         ids=lambda c: "em%d-dir%d-k%d-%s%d-B%d-%gx%g" % (*c[:3], *c[3], c[4], *c[7:]))
def test_bounded_block_pass_decides_from_bounds(bdc, case):  # noqa: F811
    em, chunk, k, (kind, s), block, h, w, level, sharp = case
    psf = synth.gaussian_psf(max(0.5, (s - 1) / 8.0), s) if kind == "gauss" else synth.airy_psf_matched(s / 10.0, s)
    img, cam = lattice_frame(h, w, k, psf, 11 + s + h, em, level, sharp)
    S = twins(bdc, img, cam, psf, bdc.BDC_SCHED_BLOCK, block, 2, 5 + s, 3, camera=em, object_sub=k,
              prior_kind=bdc.BDC_PRIOR_DIRICHLET if chunk else bdc.BDC_PRIOR_FLAT)[0]
    side = 2 * ((s // 2 + k - 1) // k) + 1                   # the footprint in pixels
    assert S.schedule_info()[2] <= side
    evals, direct, anchors = work_of(S, 4)
    if em and k == 1 and side >= 37:
        assert anchors == 0 and direct == 0                  # that pass forms no series and counts every term as one
    else:
        assert anchors > 0 and 0 <= direct < 0.5 * evals
