"""A chain's means do not depend on how many chains share the launch or on batching.

Means are FP64 sums rounded to FP32; another order of the sum is another rounding now and then.  Here the
order is made visible: at marked pixels the four PSF columns contribute 1, 2^-24, 2^-53 and 2^-53, where
the first two are a tie of FP32 and each of the last two is lost when it is added alone, but not their sum.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bdc():
    import torch
    torch.cuda.set_device(0)
    import paper_2411_00991_amd as m
    return m


PSF = np.zeros((7, 7), np.float32)
PSF[3, ::2] = 0.25


def marked(h, w):
    rho = np.full((h, w), 1e-37, np.float32)
    rho[:, 8::16] = 4.0
    rho[:, 10::16] = 4.0 * 2.0 ** -24
    rho[:, 12::16] = 4.0 * 2.0 ** -53
    rho[:, 14::16] = 4.0 * 2.0 ** -53
    return rho


def sampler(bdc, h, w, chains):
    S = bdc.Sampler(PSF, np.float32(2.0), np.float32(100.0), np.float32(1.5), height=h, width=w, n_chains=chains,
                    schedule=bdc.BDC_SCHED_BLOCK9_SERIES, max_sweeps=4, log_step0=-60.0)   # (moves of no size)
    S.init(np.full((h, w), 102.0, np.float32), np.repeat(marked(h, w)[None], chains, 0))
    return S


def at_marks(mu, w):
    return mu[..., 11:w - 4:16]


@pytest.mark.parametrize("h,w,chains", [(64, 64, 1), (256, 256, 2), (512, 512, 1), (512, 512, 4), (1024, 1024, 1), (520, 2048, 2)])
def test_one_order_at_every_size(bdc, h, w, chains):
    S = sampler(bdc, h, w, chains)
    mu = S.mu()
    S.close()
    assert np.all(at_marks(mu, w) == np.float32(1.0))


def test_batch_and_single_tiles_share_the_order(bdc):
    shapes = [(1024, 1024, 1), (512, 512, 4), (128, 96, 1)]
    alone = [sampler(bdc, *sh) for sh in shapes]
    tiles = [sampler(bdc, *sh) for sh in shapes]
    for S in alone:
        S.sweep(1)
    b = bdc.Batch(tiles)
    b.sweep(1)
    for S, T, (h, w, _) in zip(alone, tiles, shapes):
        mu, mt = S.mu(), T.mu()
        assert np.array_equal(mu, mt)
        assert np.all(at_marks(mu, w) == np.float32(1.0))
    b.close()
    for S in alone + tiles:
        S.close()
