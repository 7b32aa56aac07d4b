"""The surrogate network's kernels at the edges of their row blocks and parts (16,
32 and 64 rows to a block, whole 64-row groups, parts of 128 rows, the largest
number of parts), against the FP64 reference with the same bfloat16 rounding points
and the bars of test_gpu_mlp.py."""
import numpy as np
import pytest
import torch

import paper_1505_07674_amd as lensed
from oracle import mlp as ref

from test_gpu_mlp import NAMES, dev, problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [2, 16, 63, 64, 65, 8192, 8193, 16385])
def test_forward_at_row_block_edges(B):
    theta, norm, x, _ = problem(B)
    y = lensed.mlp_forward(dev(theta), dev(norm), dev(x)).cpu().numpy().astype(np.float64)
    yr = ref.forward(theta, norm, x, emulate_bf16=True)
    assert np.linalg.norm(y - yr) <= 1e-2 * np.linalg.norm(yr - yr.mean())


@pytest.mark.parametrize("B", [1, 15, 65, 127, 128, 257, 4097, 8193])
def test_gradient_and_step_at_part_edges(B):
    theta, norm, x, y = problem(B)
    tp, tn, tx, ty = dev(theta), dev(norm), dev(x), dev(y)
    loss, g = lensed.mlp_grad(tp, tn, tx, ty)
    lr_, gr = ref.loss_and_grad(theta, norm, x, y, emulate_bf16=True)
    assert float(loss.cpu()) == pytest.approx(lr_, rel=1e-3)
    Wg, bg = ref.unflatten(g.cpu().numpy().astype(np.float64))
    Wr, br = ref.unflatten(gr)
    for name, a, b in zip(NAMES, [t for pair in zip(Wg, bg) for t in pair], [t for pair in zip(Wr, br) for t in pair]):
        assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b), name
    # the fused step is the gradient followed by Adam: the same arithmetic, bit for bit
    m = torch.full_like(tp, 1e-3)
    v = torch.full_like(tp, 1e-5)
    p2, m2, v2 = tp.clone(), m.clone(), v.clone()
    l2 = lensed.mlp_train_step(p2, m2, v2, 7, tn, tx, ty, 1e-3)
    p1 = tp.clone()
    lensed.mlp_adam(p1, g, m, v, 7, 1e-3)
    assert torch.equal(loss, l2) and torch.equal(m, m2) and torch.equal(v, v2) and torch.equal(p1, p2)
