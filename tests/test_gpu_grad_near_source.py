"""A cuspy source right behind the lens centre, with a subsample exactly on that centre: the
re-traced subsample's partials take the deflection that it has there, none, also at the odd
N whose abscissae in the float32 part of the gradient miss the centre by a rounding. Against
the oracle, 1e-4 of the norm (test_gpu_grad.py), partial by partial for the lens's, which a
source's steep gradient times a deflection of theta_E would swamp."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks

from helpers import f32
from test_gpu_grad import oracle_grads, small_spec

pytestmark = pytest.mark.gpu
RADII = [0.0, 1e-7, 1e-5, 1e-3, 0.01, 0.02]   # arcsec, inside the re-traced radius


def to(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to("cuda:0")


@pytest.mark.parametrize("n", [1.5, 4.0])
@pytest.mark.parametrize("N,rule", [(3, "sub"), (4, "sub"), (5, "sub"), (9, "sub"), (1, "g3k7")])
def test_source_behind_the_lens_centre(N, rule, n):
    spec = small_spec(H=31, W=29, N=N, center=(0.0, 0.0))
    rng = np.random.default_rng(5)
    data, weight = rng.uniform(0, 2, (31, 29)).astype(np.float32), rng.uniform(0.5, 2, (31, 29)).astype(np.float32)
    gs = lensed.System(to(spec.psf), to(data), to(weight), pixscale=spec.pixscale, nsub=N, rule=rule)
    osys = oracle.System(31, 29, f32(spec.pixscale), N, spec.psf.astype(np.float64), data.astype(np.float64),
                         weight.astype(np.float64), rule=None if rule == "sub" else rule)
    pts = mocks.points(spec, len(RADII), seed=11).astype(np.float32)
    pts[:, 5], pts[:, 7], pts[:, 14] = 0.01, 0.5, n   # a faint, flat lens light
    pts[:, 10], pts[:, 11] = np.multiply(RADII, 0.8), np.multiply(RADII, 0.6)
    _, g = lensed.loglike_grad(to(pts), gs)
    g = g.cpu().numpy().astype(np.float64)
    _, want = oracle_grads(osys, pts)
    rel = np.linalg.norm(g - want, axis=1) / np.linalg.norm(want, axis=1)
    lens = np.linalg.norm((g - want)[:, :5], axis=1) / np.linalg.norm(want[:, :5], axis=1)
    print(f"N = {N}, {rule}, n = {n}: norm {rel.max():.1e}, lens partials {lens.max():.1e}", flush=True)
    assert np.all(rel <= 1e-4) and np.all(lens <= 1e-3)


@pytest.mark.parametrize("N,rule", [(1, "sub"), (3, "sub"), (1, "g3k7")])
def test_source_exactly_behind(N, rule):
    """The source at the origin itself, many lenses: float32 leaves the subsample on the lens
    centre 1e-7 arcsec off the source or none, as the axis ratio rounds, and a slope taken
    there would leave its rounding in the sums."""
    spec = small_spec(H=15, W=17, N=N, center=(0.0, 0.0))
    rng = np.random.default_rng(6)
    data, weight = rng.uniform(0, 2, (15, 17)).astype(np.float32), rng.uniform(0.5, 2, (15, 17)).astype(np.float32)
    gs = lensed.System(to(spec.psf), to(data), to(weight), pixscale=spec.pixscale, nsub=N, rule=rule)
    osys = oracle.System(15, 17, f32(spec.pixscale), N, spec.psf.astype(np.float64), data.astype(np.float64),
                         weight.astype(np.float64), rule=None if rule == "sub" else rule)
    pts = mocks.points(spec, 60, seed=12).astype(np.float32)
    pts[:, 1] = np.linspace(0.1, 0.99, 60)
    pts[:, 5], pts[:, 7], pts[:, 10:12], pts[:, 14] = 0.01, 0.5, 0.0, 1.5 + np.arange(60) % 4
    _, g = lensed.loglike_grad(to(pts), gs)
    g = g.cpu().numpy().astype(np.float64)
    _, want = oracle_grads(osys, pts)
    rel = np.linalg.norm(g - want, axis=1) / np.linalg.norm(want, axis=1)
    print(f"N = {N}, {rule}: {rel.max():.1e} at q = {pts[np.argmax(rel), 1]:.3f}", flush=True)
    assert np.all(rel <= 1e-4)


@pytest.mark.parametrize("theta_E", [0.0, None])
@pytest.mark.parametrize("N,rule", [(1, "sub"), (2, "sub"), (1, "g3k7")])
def test_exponential_source_on_a_subsample(N, rule, theta_E):
    """n <= 1, which is not re-traced: the light at the source's centre has a kink, and float32
    leaves the subsample that lies on it anywhere within a rounding. It then has no slope. On the
    subsample without a lens; behind the lens centre, where there is no deflection, with one."""
    spec = small_spec(H=15, W=17, N=N, pixscale=0.0625, center=(0.0, 0.0))  # pixels exact in float32
    if theta_E is None and N == 2:
        pytest.skip("no subsample on the lens centre")
    rng = np.random.default_rng(6)
    data, weight = rng.uniform(0, 2, (15, 17)).astype(np.float32), rng.uniform(0.5, 2, (15, 17)).astype(np.float32)
    gs = lensed.System(to(spec.psf), to(data), to(weight), pixscale=spec.pixscale, nsub=N, rule=rule)
    osys = oracle.System(15, 17, f32(spec.pixscale), N, spec.psf.astype(np.float64), data.astype(np.float64),
                         weight.astype(np.float64), rule=None if rule == "sub" else rule)
    pts = mocks.points(spec, 60, seed=12).astype(np.float32)
    pts[:, 1] = np.linspace(0.1, 0.99, 60)
    pts[:, 5], pts[:, 7], pts[:, 13] = 0.01, 0.5, 0.1
    pts[:, 14] = np.array([0.9, 0.95, 1.0])[np.arange(60) % 3]
    if theta_E is None:
        pts[:, 10:12] = 0.0
    else:
        pts[:, 0], pts[:, 3] = 0.0, 0.0
        k = rng.integers(-5, 6, (60, 2)) + (0.25 if N == 2 else 0.0)
        pts[:, 10:12] = k.astype(np.float32) * np.float32(spec.pixscale)
    _, g = lensed.loglike_grad(to(pts), gs)
    _, want = oracle_grads(osys, pts)
    rel = np.linalg.norm(g.cpu().numpy().astype(np.float64) - want, axis=1) / np.linalg.norm(want, axis=1)
    worst = int(np.argmax(rel))
    print(f"N = {N}, {rule}, theta_E = {theta_E}: {rel[worst]:.1e} at q = {pts[worst, 1]:.3f}, n = {pts[worst, 14]:.2f}", flush=True)
    assert np.all(rel <= 1e-4)
