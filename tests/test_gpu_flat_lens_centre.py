"""Very flat lenses with a subsample exactly on the lens centre, where the deflection is
0: the products under the reciprocals of the SIE's closed forms go with q^3 there and
must not leave the normal range. Axis ratios far below those of real lenses, down to the
smallest that validation accepts (any 0 < q <= 1), against the oracle at the bars of
test_gpu_model.py (images, 1e-6 of the peak) and test_gpu_model_grad.py (1e-4 of the
norm). Below q = 1e-6 the oracle's own atanh reaches infinity off the centre; the results
have to be finite."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks

from helpers import f32
from test_gpu_grad import gpu_system, oracle_grads, small_obs, small_spec
from test_gpu_model import gsys, models, osys
from test_gpu_model_grad import fd_grad, mock

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def to(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# one lens at the origin, shear, a foreground and a lensed Sersic, sky
def general_point(q):
    return np.array([0, 0, 0.6, q, 0.7, 0.03, 0.4, 0.1, 0.05, 1.0, 0.5, 2.0, 0.8, 0.3, 0.05, -0.02, 0.9, 0.3, 1.5, 0.7,
                     1.1, 0.2], np.float32)


@pytest.mark.parametrize("q", [0.05, 2e-3, 1e-3, 1e-4, 1e-6, 1e-9, 1e-20, 1e-38, 1.4e-45])
def test_general_model(q):
    print(f"general model, q = {q}", flush=True)
    gm, om = models(1, ["foreground", "lensed"], shear=True, sky=True)
    spec = small_spec(H=35, W=33, N=3, center=(0.0, 0.0))   # odd sides and N: a subsample on the origin
    t = general_point(q)
    img = lensed.render_model(to(t), gsys(spec), gm).cpu().numpy().astype(np.float64)
    assert np.isfinite(img).all()
    if q >= 1e-6:
        want = oracle.render_model(osys(spec), om, t.astype(np.float64))
        assert np.max(np.abs(img - want)) <= 1e-6 * np.max(want)
    data, weight = mock(spec, om, general_point(0.7))
    ll, g = lensed.loglike_model_grad(to(t[None]), gsys(spec, data, weight), gm)
    assert torch.isfinite(ll).all()
    if q >= 1e-9:   # below, 1/q^2 leaves the range in which the partials mean anything
        assert torch.isfinite(g).all()
    if q >= 1e-4:
        want = fd_grad(osys(spec, data.astype(np.float64), weight.astype(np.float64)), om, t)
        keep = np.ones(len(t), bool)
        keep[:2] = False   # the surface brightness has a kink at a subsample on the lens centre
        got = g.cpu().numpy().astype(np.float64)[0]
        assert np.linalg.norm((got - want)[keep]) <= 1e-4 * np.linalg.norm(want[keep])


@pytest.mark.parametrize("q", [0.05, 2e-3, 1e-3, 5e-4])
def test_retraced_centre(q):
    """A cuspy source at the origin: the subsample on the lens centre is re-traced in float64."""
    print(f"re-traced centre, q = {q}", flush=True)
    spec = small_spec(H=31, W=29, N=1, center=(0.0, 0.0))
    t = mocks.points(spec, 1, seed=5)[0].astype(np.float32)
    t[1], t[10:12], t[14] = q, 0.0, 4.0
    img = lensed.render(to(t), gpu_system(spec, small_obs(spec)))
    assert torch.isfinite(img).all()


@pytest.mark.parametrize("rule", ["sub", "g3k7"])
def test_gradient_17_parameters(rule):
    """The float32 gradient, whose psi^2 = q^2 (x'^2 + tiny) at the centre has to be a normal
    float32 too; 1e-4 of the oracle's norm (test_gpu_grad.py)."""
    qs = [0.05, 1e-2, 1e-3, 4e-4, 3e-4, 1e-4, 5e-5, 1e-5, 1e-6, 1e-9, 1e-13, 1e-30]
    spec = small_spec(H=31, W=29, N=1, center=(0.0, 0.0))
    obs = small_obs(spec)
    pts = mocks.points(spec, len(qs), seed=5).astype(np.float32)
    pts[:, 1] = qs
    gs = lensed.System(to(spec.psf), to(obs.data), to(obs.weight), pixscale=spec.pixscale, nsub=1, rule=rule)
    o = oracle.System(spec.height, spec.width, f32(spec.pixscale), 1, spec.psf.astype(np.float64),
                      obs.data.astype(np.float64), obs.weight.astype(np.float64),
                      rule=None if rule == "sub" else rule)
    _, g = lensed.loglike_grad(to(pts), gs)
    g = g.cpu().numpy().astype(np.float64)
    _, want = oracle_grads(o, pts)
    for i, q in enumerate(qs):
        if q >= 1e-6:
            rel = np.linalg.norm(g[i] - want[i]) / np.linalg.norm(want[i])
            print(f"rule {rule}, q = {q}: relative gradient error {rel:.1e}", flush=True)
            assert rel <= 1e-4
        elif q >= 1e-19:   # below, 1/q^2 is no float32
            assert np.isfinite(g[i]).all(), q
