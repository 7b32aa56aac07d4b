"""The per-point constants at the edges of their tables and tiles: Sersic indices at
the ends of the accepted range and next to the joints of the b_n polynomials, points
that fill a block of the prologue only in part, and PSFs from one tap to the largest
side (normalisation and the border tables of the gradient, by every border class).
Images to 1e-5 of the peak (the forward parity bar), gradients to 1e-4 of the norm
(test_gpu_grad.py)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks

from helpers import oracle_system
from test_gpu_grad import check, small_obs, small_spec

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
UP, DOWN = np.float32(1 + 2e-7), np.float32(1 - 2e-7)
JOINTS = [np.float32(v) for v in (0.25, 0.5, 0.75, 1.0, 1.25, 2.0, 3.5, 4.0, 7.0, 8.0)]
INDICES = [np.float32(0.2), np.float32(10.0)] + [j * s for j in JOINTS for s in (DOWN, np.float32(1), UP)]


@pytest.mark.parametrize("magnitude", [False, True])
def test_sersic_indices_at_the_joints(magnitude):
    spec = small_spec(H=33, W=30)
    pts = mocks.points(spec, len(INDICES), seed=7).astype(np.float32)
    pts[:, 7], pts[:, 14] = INDICES, INDICES[::-1]
    osys = oracle_system(spec)
    kw = dict(amplitude="magnitude", zero_point=2.0) if magnitude else {}
    gsys = lensed.System(torch.from_numpy(spec.psf).to(DEV), pixscale=spec.pixscale, nsub=spec.nsub,
                         height=spec.height, width=spec.width,
                         center=(spec.center_x, spec.center_y), **kw)
    for t in pts:
        ref = t.astype(np.float64)
        if magnitude:
            t[5], t[12] = 1.0, 2.0
            ref = t.astype(np.float64)
            for k in (5, 12):
                ref[k] = oracle.intensity_from_magnitude(ref[k], ref[k + 1], ref[k + 2], 2.0)
        print(f"n = {t[7]!r}, {t[14]!r}", flush=True)
        img = lensed.render(torch.from_numpy(t).to(DEV), gsys).cpu().numpy().astype(np.float64)
        want = oracle.render(osys, ref)
        assert np.max(np.abs(img - want)) <= 1e-5 * np.max(np.abs(want))


@pytest.mark.parametrize("points", [1, 7, 9])
def test_points_that_fill_a_block_in_part(points):
    spec = small_spec(H=24, W=22)
    obs = small_obs(spec)
    pts = mocks.points(spec, points, seed=50 + points)
    pts[-1, 14] = 1.25   # a joint of the b_n polynomials, where db_n/dn changes piece
    check(spec, obs, pts, loglike_bar=False)


@pytest.mark.parametrize("ph,pw", [(1, 1), (1, 5), (9, 1), (3, 17), (63, 63)])
def test_psf_sides(ph, pw):
    rng = np.random.default_rng(ph * 64 + pw)
    psf = rng.uniform(0.1, 1.0, (ph, pw)) * np.exp(-np.add.outer(np.linspace(-2, 2, ph) ** 2 if ph > 1 else [0.0],
                                                                 np.linspace(-2, 2, pw) ** 2 if pw > 1 else [0.0]))
    spec = small_spec(H=37, W=41, psf=psf)
    spec.mask = np.ones_like(spec.mask)   # every border pixel counts
    obs = small_obs(spec)
    check(spec, obs, mocks.points(spec, 3, seed=60), loglike_bar=False)
