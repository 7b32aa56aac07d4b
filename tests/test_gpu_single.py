"""One image at a time: the kernel that renders and corrects in one pass and the PSF
kernel that adds its own tile sums, against the batch (the list of flagged waves and a
summing launch of its own) and the oracle, at image sizes around their blocks and tiles
and around the largest they take, for a cuspy source (corrected subsamples) and a flat
one, and again on the same buffers (the block counter starts over). log L equals the
batch's to its summation order, 1e-12 (test_gpu_grad.py); with a 21 x 21 PSF the batch's
compensated chains have eight rows, not four, which round a group's first product
differently, and the forward parity bar applies."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks

from helpers import loglike_tolerance, oracle_system
from test_gpu_grad import gpu_system, small_obs, small_spec

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def points(spec, seed):
    pts = mocks.points(spec, 3, seed=seed).astype(np.float32)
    pts[0, 14], pts[1, 14], pts[2, 14] = 4.0, 0.8, 2.5
    pts[0, 10:12] = 0.02   # a cuspy source near the caustic: many corrected pixels
    return pts


@pytest.mark.parametrize("h,w,N,psf", [(1, 1, 1, 1), (8, 16, 2, 7), (16, 16, 8, 21), (17, 15, 9, 5), (63, 65, 4, 21),
                                       (128, 128, 2, 7), (129, 128, 3, 9)])
def test_one_image_equals_the_batch(h, w, N, psf):
    spec = small_spec(H=h, W=w, N=N, psf=mocks.moffat_psf(psf, 0.15, 3.0, 0.08) if psf > 1 else np.ones((1, 1)))
    spec.mask = np.ones_like(spec.mask)
    obs = small_obs(spec)
    gsys, osys = gpu_system(spec, obs), oracle_system(spec, obs)
    pts = points(spec, h + w)
    tp = torch.from_numpy(pts).to(DEV)
    batch = lensed.loglike_batch(tp, np.zeros(3, np.int32), [gsys]).cpu().numpy()
    for rep in range(3):
        for i in range(3):
            one = float(lensed.loglike(tp[i], gsys))
            bar = 1e-12 * abs(batch[i]) if psf != 21 else loglike_tolerance(batch[i], obs.weight)
            assert abs(one - batch[i]) <= bar
    for i in range(3):
        img = lensed.render(tp[i], gsys).cpu().numpy().astype(np.float64)
        want = oracle.render(osys, pts[i].astype(np.float64))
        assert np.max(np.abs(img - want)) <= 1e-5 * np.max(np.abs(want))


@pytest.mark.parametrize("h,w", [(512, 512), (513, 512)])
def test_the_largest_single_image(h, w):
    """Both sides of the size that the one-pass kernels take; only log L, against the batch."""
    spec = small_spec(H=h, W=w, N=1, pixscale=0.02)
    psf = torch.from_numpy(spec.psf).to(DEV)
    rng = np.random.default_rng(h)
    data = torch.from_numpy(rng.uniform(0, 1, (h, w)).astype(np.float32)).to(DEV)
    gsys = lensed.System(psf, data, torch.ones_like(data), pixscale=0.02, nsub=1)
    tp = torch.from_numpy(points(spec, 3)).to(DEV)
    batch = lensed.loglike_batch(tp, np.zeros(3, np.int32), [gsys]).cpu().numpy()
    for i in range(3):
        assert abs(float(lensed.loglike(tp[i], gsys)) - batch[i]) <= 1e-12 * abs(batch[i])


def test_both_sides_of_the_fused_render():
    """64 points of 64 x 64 pixels are 4096 waves, the most that correct their own pixels
    as they render; a 65th point takes the list and its kernel. The same log L, and the
    same gradient to the order of the corrections' sums (both in float64: 1e-6 of the norm)."""
    spec = small_spec(H=64, W=64)
    obs = small_obs(spec)
    pts = mocks.points(spec, 65, seed=11).astype(np.float32)
    pts[::2, 14] = 3.5   # cuspy sources
    tp = torch.from_numpy(pts).to(DEV)
    gsys = gpu_system(spec, obs)
    ll64, g64 = lensed.loglike_grad(tp[:64].contiguous(), gsys)
    ll65, g65 = lensed.loglike_grad(tp, gsys)
    assert torch.equal(ll64, ll65[:64])
    assert torch.all((g64 - g65[:64]).norm(dim=1) <= 1e-6 * g64.norm(dim=1))
