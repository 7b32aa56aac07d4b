"""General models at the edges of their kernels: axis ratios on both sides of the
choice between the closed form and the series in 1 - q^2, round and very flat
lenses, subsamples exactly on a lens and a light centre, odd and even numbers of
subsamples per row, and numbers of components around what one gradient pass takes
(two SIEs, two Sersics). Images to the bar of test_gpu_model.py (1e-6 of the peak),
gradients to that of test_gpu_model_grad.py (1e-4 of the norm)."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_1505_07674_amd as lensed

from test_gpu_grad import small_spec
from test_gpu_model import gsys, models, osys
from test_gpu_model_grad import fd_grad, mock

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
Q_EDGE = math.sqrt(1 - 0.05)   # where 1 - q^2 = 0.05


def points(n, seed, qs, planes, shear, sky, centred):
    rng = np.random.default_rng(seed)
    rows = []
    for _ in range(n):
        p = []
        for k, q in enumerate(qs):
            c = (0.0, 0.0) if centred and k == 0 else tuple(rng.uniform(-0.4, 0.4, 2))
            p += [*c, rng.uniform(0.2, 0.9), q, rng.uniform(0, math.pi)]
        if shear:
            p += [rng.uniform(0.01, 0.08), rng.uniform(0, math.pi)]
        for j, plane in enumerate(planes):
            c = (0.0, 0.0) if centred and j == 0 else tuple(rng.uniform(-0.3, 0.3, 2))
            p += [*c, rng.uniform(0.2, 1.5), rng.uniform(0.2, 0.8), rng.uniform(0.6, 4), rng.uniform(0.4, 0.98),
                  rng.uniform(0, math.pi)]
        if sky:
            p += [rng.uniform(0.05, 0.5)]
        rows.append(p)
    return np.array(rows, np.float32)


F, S = "foreground", "lensed"
CASES = [   # axis ratios, planes, shear, sky, N, centred
    ([Q_EDGE - 1e-4, Q_EDGE + 1e-4], [F, S], True, True, 2, False),
    ([1.0], [S], True, False, 3, True),
    ([1.0 - 1e-6, 0.05], [F, S, S], False, True, 1, False),
    ([0.7], [F], False, False, 5, True),
    ([], [S], True, True, 4, False),
    ([], [F, F, F], False, False, 3, True),
    ([0.8, 0.99, 0.3], [S, F, S, F, S], True, True, 3, True),
    ([0.6] * 8, [F, S] * 4, True, True, 2, False),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_images_and_gradients_at_the_edges(case):
    qs, planes, shear, sky, N, centred = CASES[case]
    spec = small_spec(H=35, W=33, N=N, center=(0.0, 0.0))   # odd sides: a pixel centred on the origin
    gm, om = models(len(qs), planes, shear=shear, sky=sky)
    pts = points(2, 90 + case, qs, planes, shear, sky, centred)
    print(f"general model edges: {len(qs)} SIEs (q {qs}), {len(planes)} Sersics, N = {N}", flush=True)
    for t in pts:
        img = lensed.render_model(torch.from_numpy(t).to(DEV), gsys(spec), gm).cpu().numpy().astype(np.float64)
        ref = oracle.render_model(osys(spec), om, t.astype(np.float64))
        assert np.max(np.abs(img - ref)) <= 1e-6 * np.max(np.abs(ref))
    if 1.0 in qs:   # the oracle's central difference would step past q = 1
        return
    # the mock's truth lies away from the points, so that the gradient is not noise
    truth = points(1, 190 + case, qs, planes, shear, sky, False)[0]
    data, weight = mock(spec, om, truth)
    g, o = gsys(spec, data, weight), osys(spec, data.astype(np.float64), weight.astype(np.float64))
    if any(q > 1 - 1e-4 for q in qs):
        pts[:, 3] = 0.999   # a difference step within (0, 1]
    _, gg = lensed.loglike_model_grad(torch.from_numpy(pts).to(DEV), g, gm)
    gg = gg.cpu().numpy().astype(np.float64)
    for i, t in enumerate(pts):
        want = fd_grad(o, om, t)
        if centred:   # the surface brightness has a kink at a subsample on a centre: leave the centres out
            keep = np.ones(len(want), bool)
            keep[:2] = not len(qs)
            o0 = 5 * len(qs) + (2 if shear else 0)
            keep[o0:o0 + 2] = False
        else:
            keep = slice(None)
        assert np.linalg.norm((gg[i] - want)[keep]) <= 1e-4 * np.linalg.norm(want[keep])
