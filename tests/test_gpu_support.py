"""The gradient's support (the pixels within the PSF box of a weighted one) at the
edges of its 64-pixel words, 512-pixel segments, bands and tiles: widths around them,
odd and even (one or two pixels per render unit), PSFs from one tap to wide ones, and
weights on a few pixels, in the corners, at the joints or nowhere. Gradients against
the oracle, log L against the batch (test_gpu_grad.py); the gradients to 1e-3 of the
norm: a pixel's float32 error, up to 1e-5 of the peak, is not averaged here, and the
residuals of these pixels are from 1e-2 of the peak."""
import numpy as np
import pytest
import torch

import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks

from test_gpu_grad import check, gpu_system, small_obs, small_spec

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def sparse(spec, pixels):
    """A mock observation with weights on the given pixels alone."""
    spec.mask = np.ones_like(spec.mask)
    obs = small_obs(spec)
    keep = np.zeros_like(obs.weight)
    for r, c in pixels:
        keep[r, c] = 1.0
    obs.weight = (obs.weight * keep).astype(np.float32)
    return obs


@pytest.mark.parametrize("h,w,ph,pw,pixels", [
    (9, 63, 7, 7, [(0, 62), (8, 0), (4, 30)]),
    (9, 64, 7, 7, [(0, 63), (8, 0), (4, 31)]),
    (17, 65, 1, 1, [(7, 64), (8, 63), (16, 0), (8, 40)]),
    (24, 130, 5, 31, [(7, 63), (8, 64), (15, 127), (16, 128), (12, 70)]),
    (8, 514, 7, 3, [(3, 255), (4, 260), (0, 511), (7, 512), (2, 513)]),
    (7, 1030, 3, 63, [(3, 511), (3, 512), (6, 1029), (0, 500), (2, 530)]),
    (70, 33, 31, 5, [(0, 0), (69, 32), (35, 16), (40, 20)]),
    (40, 1, 9, 9, [(20, 0), (7, 0), (31, 0)]),
])
def test_sparse_weights(h, w, ph, pw, pixels):
    rng = np.random.default_rng(h * w)
    spec = small_spec(H=h, W=w, psf=rng.uniform(0.2, 1.0, (ph, pw)), center=(0.01, -0.02))
    obs = sparse(spec, pixels)
    check(spec, obs, mocks.points(spec, 3, seed=h + w), tol=1e-3, loglike_bar=False)


def test_no_weighted_pixel():
    spec = small_spec(H=20, W=70)
    obs = sparse(spec, [])
    pts = torch.from_numpy(mocks.points(spec, 2, seed=1)).to(DEV)
    ll, g = lensed.loglike_grad(pts, gpu_system(spec, obs))
    assert torch.all(ll == 0) and torch.all(g == 0)
