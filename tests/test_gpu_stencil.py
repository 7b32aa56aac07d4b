"""The PSF stencil on the matrix cores (Eq. 15) and its transpose over PSF shapes
and image shapes: every count of matrix steps, kernels that are no square, tiles
with ragged rows and columns, single images and batches, and tiles with a
non-finite value. The reference convolves the library's own unconvolved image in
float64, so the tolerance is the a-priori bound of a float32 dot product of n
terms with rounded taps, n u / (1 - n u) times the sum of |tap x value|, with
n = taps + 1 and u = 2^-24."""
import numpy as np
import pytest
import torch
from scipy import ndimage

import oracle
import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks
from paper_1505_07674_amd.binding import Context

from helpers import oracle_system

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
U = 2.0 ** -24

# (height, width, PSF height, PSF width)
SHAPES = [(37, 53, 1, 1), (41, 47, 3, 3), (33, 66, 5, 5), (64, 64, 7, 7), (50, 51, 9, 9), (87, 101, 11, 11),
          (40, 70, 13, 13), (61, 49, 15, 15), (45, 80, 17, 17), (55, 43, 19, 19), (72, 90, 21, 21), (52, 60, 23, 23),
          (39, 77, 25, 25), (48, 48, 27, 27), (66, 35, 33, 33), (59, 71, 35, 35), (70, 70, 49, 49), (57, 58, 51, 51),
          (75, 69, 63, 63), (36, 84, 3, 21), (84, 36, 21, 3), (30, 64, 63, 1), (64, 30, 1, 63), (5, 7, 21, 21),
          (1, 130, 9, 5), (130, 1, 5, 9)]


def _psf(ph, pw, rng):
    return (rng.random((ph, pw)) ** 2 + 0.01).astype(np.float32)


def _convolved(img, psf):
    f = psf.astype(np.float64)
    f = f / f.sum()
    return (ndimage.convolve(img.astype(np.float64), f, mode="nearest"),
            ndimage.convolve(np.abs(img.astype(np.float64)), f, mode="nearest"))


@pytest.mark.parametrize("H,W,ph,pw", SHAPES)
def test_convolution_and_loglike_over_psf_shapes(H, W, ph, pw):
    rng = np.random.default_rng(H * 1000 + W + ph * 7 + pw)
    psf = _psf(ph, pw, rng)
    pts = mocks.points(mocks.c1_spec(), 3, seed=H + ph)
    print(f"stencil {H}x{W}, PSF {ph}x{pw}", flush=True)
    data = rng.standard_normal((H, W)).astype(np.float32)
    weight = (rng.random((H, W)) * (rng.random((H, W)) < 0.7)).astype(np.float32)
    gs = lensed.System(torch.from_numpy(psf).to(DEV), torch.from_numpy(data).to(DEV), torch.from_numpy(weight).to(DEV),
                       pixscale=0.05, nsub=2)
    tp = torch.from_numpy(pts).to(DEV)
    n = ph * pw + 1
    gamma = n * U / (1 - n * U)
    ref, bound = [], []
    for t in tp:
        raw = lensed.render(t, gs, apply_psf=False).cpu().numpy()
        img = lensed.render(t, gs).cpu().numpy()
        want, mag = _convolved(raw, psf)
        d = gamma * mag
        assert np.all(np.abs(img - want) <= d + 1e-45), np.max(np.abs(img - want) / (d + 1e-45))
        r, w = data.astype(np.float64) - want, weight.astype(np.float64)
        ref.append(-0.5 * np.sum(w * r * r))
        # L* within d, the residual and the weighted residual rounded once each, the
        # product once
        dr = d + 2 * U * (np.abs(data) + np.abs(want) + d)
        bound.append(0.5 * np.sum(w * (2 * np.abs(r) * dr + dr * dr) + 4 * U * w * (np.abs(r) + dr) ** 2))
    ctx = Context(0)
    sop = np.zeros(3, np.int32)
    one = np.array([lensed.loglike(t, gs, ctx=ctx).item() for t in tp])
    many = lensed.loglike_batch(tp, sop, [gs], ctx=ctx).cpu().numpy()
    masked = lensed.loglike_batch(tp, sop, [gs], ctx=ctx, masked=True).cpu().numpy()
    ctx.close()
    for ll in (one, many, masked):
        assert np.all(np.abs(ll - np.array(ref)) <= np.array(bound)), (ll, ref, bound)


@pytest.mark.parametrize("P,H,W", [(7, 70, 75), (11, 61, 90), (21, 90, 101), (31, 80, 66)])
def test_non_finite_pixels_reach_their_psf_box_and_no_further(P, H, W):
    """A source bright enough to overflow: the convolved image is non-finite
    exactly where the PSF box holds a non-finite pixel."""
    psf = _psf(P, P, np.random.default_rng(P))
    t = mocks.c1_spec().truth.copy()
    t[12], t[13], t[14] = 3e38, 0.1, 3.9
    gs = lensed.System(torch.from_numpy(psf).to(DEV), pixscale=0.05, nsub=2, height=H, width=W)
    tp = torch.from_numpy(t).to(DEV)
    raw = lensed.render(tp, gs, apply_psf=False).cpu().numpy()
    img = lensed.render(tp, gs).cpu().numpy()
    bad = ~np.isfinite(raw)
    assert 0 < bad.sum() < bad.size / 4
    reach = ndimage.maximum_filter(bad.astype(np.uint8), size=(P, P), mode="nearest") > 0
    print(f"stencil {H}x{W}, PSF {P}x{P}: {bad.sum()} non-finite pixels reach {reach.sum()}", flush=True)
    far = img[~reach]
    assert np.all(np.isfinite(far) | (np.abs(far) > 1e38))
    assert not np.any(np.isnan(far)) and not np.any(np.isfinite(img[reach]))


@pytest.mark.parametrize("H,W,ph,pw", [(40, 44, 13, 13), (37, 50, 25, 25), (43, 39, 31, 5), (36, 64, 5, 35)])
def test_gradient_over_psf_shapes(H, W, ph, pw):
    """The transposed stencil over kernel shapes, against the oracle's gradient."""
    rng = np.random.default_rng(ph + pw)
    base = mocks.c1_spec()
    spec = mocks.SystemSpec(f"stencil_grad_{ph}x{pw}", H, W, 2, _psf(ph, pw, rng), base.truth, base.prior,
                            mocks.annulus_mask(H, W, 0.2, 10.0, 0.08), 31, True, pixscale=0.08)
    osys = oracle_system(spec)
    obs = mocks.make_observation(spec, lambda t: oracle.render(osys, np.asarray(t, np.float64)))
    osys = oracle_system(spec, obs)
    pts = mocks.points(spec, 4, seed=ph)
    gs = lensed.System(torch.from_numpy(spec.psf).to(DEV), torch.from_numpy(obs.data).to(DEV),
                       torch.from_numpy(obs.weight).to(DEV), pixscale=spec.pixscale, nsub=spec.nsub)
    print(f"stencil gradient {H}x{W}, PSF {ph}x{pw}", flush=True)
    _, g = lensed.loglike_grad(torch.from_numpy(pts).to(DEV), gs)
    g = g.cpu().numpy().astype(np.float64)
    for k, t in enumerate(pts):
        _, want = oracle.loglike_grad(osys, t.astype(np.float64))
        assert np.linalg.norm(g[k] - want) <= 1e-4 * np.linalg.norm(want)
