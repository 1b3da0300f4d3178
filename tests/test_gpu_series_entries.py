"""The block-series scan holds up to three footprint entries per thread to side 27, four beyond and in
batches: a tile alone reaches the state that it reaches in a batch, bit for bit, on both sides of the line."""

import numpy as np
import pytest

from paper_2411_00991_amd import synth
from test_gpu_decisions import bdc, f32, frame  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [3, 15, 17, 27, 29, 31])
def test_alone_as_in_a_batch(bdc, s):  # noqa: F811
    h, w = 2 * s + 9, 2 * s + 20
    psf = synth.gaussian_psf(max(0.5, (s - 1) / 8.0), s)
    img, cam = frame(h, w, psf, 70 + s, 2.0)
    S = []
    for _ in range(2):
        S.append(bdc.Sampler(f32(psf), *[f32(a) for a in cam.maps(h, w)], height=h, width=w, n_chains=2, seed=s, burn_in=3,
                             schedule=bdc.BDC_SCHED_BLOCK_SERIES, log_step0=-0.3))
        S[-1].init(f32(img))
    S[0].sweep(5)
    b = bdc.Batch(S[1:])
    b.sweep(5)
    ra, la, _ = S[0].rho()
    rb, lb, _ = S[1].rho()
    assert np.array_equal(ra, rb) and np.array_equal(la, lb) and np.array_equal(S[0].mu(), S[1].mu())
    b.close()
