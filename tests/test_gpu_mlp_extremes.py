"""The surrogate's SiLU and its derivative far from zero: pre-activations so negative that
exp(-z) overflows (SiLU and its slope are 0 there), up to the largest float32, and inf and
NaN among the inputs (inf stays inf; NaN where the plain quotient z / (1 + exp(-z)) is
NaN). Positive weights, so that one input drives every unit of a layer
the same way; values against the FP64 reference, to the bars of test_gpu_mlp.py."""
import numpy as np
import pytest
import torch

import paper_1505_07674_amd as lensed
from oracle import mlp as ref

from test_gpu_mlp import NAMES, dev

pytestmark = pytest.mark.gpu
RNG = np.random.default_rng(23)


def network():
    Ws, bs = ref.unflatten(ref.init_params(7))
    bs = [RNG.uniform(0.02, 0.2, b.shape) for b in bs]
    theta = ref.flatten([np.abs(W) / 16 for W in Ws], bs).astype(np.float32)
    norm = np.concatenate([np.zeros(17), np.ones(17), [-0.5, 2.0]]).astype(np.float32)
    x = RNG.uniform(-1, 1, (5, 17)).astype(np.float32)
    return theta, norm, x


@pytest.mark.parametrize("value", [-75.0, -90.0, -300.0, -1e5, -1e30, 300.0, 1e20, 3e38])
def test_large_finite_pre_activations(value):
    print(f"input {value}", flush=True)
    theta, norm, x = network()
    x[2] = value
    y = lensed.mlp_forward(dev(theta), dev(norm), dev(x)).cpu().numpy().astype(np.float64)
    with np.errstate(over="ignore"):
        want = ref.forward(theta, norm, x, emulate_bf16=True)
    assert np.all(np.abs(y - want) <= 1e-2 * np.abs(want - norm[34]))
    targets = (want + 0.5 * np.arange(5)).astype(np.float32)
    loss, g = lensed.mlp_grad(dev(theta), dev(norm), dev(x), dev(targets))
    if value > 1e4:   # the squared error leaves float32
        return
    with np.errstate(over="ignore"):
        lr_, gr = ref.loss_and_grad(theta, norm, x, targets, emulate_bf16=True)
    Wg, bg = ref.unflatten(g.cpu().numpy().astype(np.float64))
    Wr, br = ref.unflatten(gr)
    if value < 0:   # the row's error is of the others' size: nothing cancels
        assert float(loss.cpu()) == pytest.approx(lr_, rel=1e-2)
        for name, a, b in zip(NAMES, [t for p in zip(Wg, bg) for t in p], [t for p in zip(Wr, br) for t in p]):
            assert np.linalg.norm(a - b) <= 2e-2 * np.linalg.norm(b), name


@pytest.mark.parametrize("value,want", [(np.inf, np.inf), (-np.inf, np.nan), (np.nan, np.nan)])
def test_infinite_inputs(value, want):
    print(f"input {value}", flush=True)
    theta, norm, x = network()
    clean = lensed.mlp_forward(dev(theta), dev(norm), dev(x)).cpu().numpy()
    x[2] = value
    y = lensed.mlp_forward(dev(theta), dev(norm), dev(x)).cpu().numpy()
    assert np.array_equal(y[2], np.float32(want), equal_nan=True)
    keep = np.arange(5) != 2
    assert np.array_equal(y[keep], clean[keep])   # the other rows of the block are their own
    loss, g = lensed.mlp_grad(dev(theta), dev(norm), dev(x), dev(np.zeros(5, np.float32)))
    assert not torch.isfinite(loss).any() and torch.isnan(g).any()
