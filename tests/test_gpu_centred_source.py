"""A cuspy source right behind the lens centre, with a subsample on that centre: the
deflection there has to be exactly 0, since the light of a Sersic source of index n goes
with R^(1/n) and turns a residue of 1e-16 into 1e-3 of the pixel. Images against the
oracle, to the bars of test_gpu_parity.py (the 17-parameter render, whose centre is
re-traced in float64: 1e-5 of the peak) and test_gpu_model.py (general models: 1e-6)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks

from helpers import oracle_system
from test_gpu_grad import gpu_system, small_obs, small_spec
from test_gpu_model import gsys, models, osys

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
QS = [1.0, 0.98, 0.7, 0.41, 0.2, 0.05, 1e-3]


def to(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("n", [1.5, 4.0, 8.0])
def test_render(q, n):
    spec = small_spec(H=31, W=29, N=1, center=(0.0, 0.0))
    t = mocks.points(spec, 1, seed=5)[0].astype(np.float32)
    t[1], t[10:12], t[14] = q, 0.0, n
    img = lensed.render(to(t), gpu_system(spec, small_obs(spec))).cpu().numpy().astype(np.float64)
    want = oracle.render(oracle_system(spec), t.astype(np.float64))
    err = np.max(np.abs(img - want)) / np.max(want)
    print(f"q = {q}, n = {n}: {err:.1e}", flush=True)
    assert err <= 1e-5


@pytest.mark.parametrize("q", QS)
@pytest.mark.parametrize("n", [1.5, 4.0, 8.0])
def test_general_model(q, n):
    gm, om = models(1, ["lensed"], shear=True)
    spec = small_spec(H=35, W=33, N=3, center=(0.0, 0.0))
    t = np.array([0, 0, 0.6, q, 0.7, 0.03, 0.4, 0, 0, 0.9, 0.3, n, 0.7, 1.1], np.float32)
    img = lensed.render_model(to(t), gsys(spec), gm).cpu().numpy().astype(np.float64)
    want = oracle.render_model(osys(spec), om, t.astype(np.float64))
    err = np.max(np.abs(img - want)) / np.max(want)
    print(f"q = {q}, n = {n}: {err:.1e}", flush=True)
    assert err <= 1e-6
