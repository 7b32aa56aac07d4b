"""The rows at the edges of the surrogate kernels' row blocks, 64-row groups and parts,
one by one: a row that is dropped, doubled or taken from its neighbour has to show, also
in a batch of thousands.

Forward: every row within 5e-2 of the predictions' spread (a wrong row is off by about
the spread itself; the operands' rounding to bfloat16, the same on both sides but for sums
that fall on the other side of a tie, moves a row by about 1e-3).
Gradient: the targets are the reference's own predictions except at one row, whose error
is 100 in normalised units, so that the loss and every gradient tensor are that row's; the
other rows' errors of about 1e-3 each add less than 1e-2 of it in the largest batch. Bars:
2e-2 of the loss and of each tensor's norm."""
import numpy as np
import pytest
import torch

import paper_1505_07674_amd as lensed
from oracle import mlp as ref

from test_gpu_mlp import NAMES, dev, problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 15, 16, 17, 63, 64, 65, 8191, 8192, 8193, 16384, 16385, 16447])
def test_every_row_of_the_forward(B):
    theta, norm, x, _ = problem(B)
    y = lensed.mlp_forward(dev(theta), dev(norm), dev(x)).cpu().numpy().astype(np.float64)
    want = ref.forward(theta, norm, x, emulate_bf16=True)
    spread = want.std() if B > 2 else norm[35]
    worst = int(np.argmax(np.abs(y - want)))
    print(f"B = {B}: worst row {worst}, {abs(y - want)[worst] / spread:.1e} of the spread", flush=True)
    assert abs(y - want)[worst] <= 5e-2 * spread


@pytest.mark.parametrize("B", [1, 15, 17, 65, 127, 128, 129, 257, 4097, 8192, 8193])
def test_single_rows_of_the_gradient(B):
    theta, norm, x, _ = problem(B)
    tp, tn, tx = dev(theta), dev(norm), dev(x)
    y0 = ref.forward(theta, norm, x, emulate_bf16=True)
    last = (B - 1) // 128 * 128   # the first row of the last 128
    for row in sorted({0, B - 1, last, max(last - 1, 0), (B - 1) // 16 * 16}):
        y = y0.copy()
        y[row] -= 100.0 * norm[35]
        y = y.astype(np.float32)
        loss, g = lensed.mlp_grad(tp, tn, tx, dev(y))
        lr_, gr = ref.loss_and_grad(theta, norm, x, y, emulate_bf16=True)
        assert float(loss.cpu()) == pytest.approx(lr_, rel=2e-2), row
        Wg, bg = ref.unflatten(g.cpu().numpy().astype(np.float64))
        Wr, br = ref.unflatten(gr)
        rel = [np.linalg.norm(a - b) / np.linalg.norm(b)
               for a, b in zip([t for p in zip(Wg, bg) for t in p], [t for p in zip(Wr, br) for t in p])]
        print(f"B = {B}, row {row}: worst tensor {NAMES[int(np.argmax(rel))]} {max(rel):.1e}", flush=True)
        assert max(rel) <= 2e-2
