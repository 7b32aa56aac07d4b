"""The measured render schedule: render and cusp corrections are timed together, and
launches that can correct their pixels as they render (at most 4096 waves, one pixel per
thread, blocks of at most 256) keep a schedule apart from larger ones over the same
shapes, in either order. Small launches are 15 % faster with the corrections in the render
kernel, a difference the timing of the schedules cannot miss; every schedule gives the
same log L bit for bit."""
import numpy as np
import pytest
import torch

import paper_1505_07674_amd as lensed
from paper_1505_07674_amd import mocks
from paper_1505_07674_amd.binding import Context

from test_gpu_grad import small_spec
from test_gpu_schedule import context_with

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
SMALL, LARGE = 16, 600


def to(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(DEV)


def system(h, w, n):
    spec = small_spec(H=h, W=w, N=n, pixscale=0.05)
    rng = np.random.default_rng(h)
    gs = lensed.System(to(spec.psf), to(rng.uniform(0, 1, (h, w))), to(rng.random((h, w)) < 0.7), pixscale=0.05, nsub=n)
    return gs, to(mocks.points(spec, LARGE, seed=9))


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("order", [(SMALL,), (SMALL, LARGE, SMALL), (LARGE, SMALL)])
@pytest.mark.parametrize("h,w,n", [(87, 101, 3), (100, 100, 4)])
def test_small_launches_keep_a_fused_schedule(h, w, n, order, masked):
    gs, pts = system(h, w, n)
    ctx = Context(0)
    for P in order:
        lensed.loglike_batch(pts[:P].contiguous(), np.zeros(P, np.int32), [gs], ctx=ctx, masked=masked)
        torch.cuda.synchronize()
        s = ctx.batch_schedule()
        print(f"{h} x {w}, N = {n}, {P} points: {s}", flush=True)
        if P == SMALL:
            assert s["render_pixels_per_thread"] == 1 and s["render_block"] <= 256
    ctx.close()


@pytest.mark.parametrize("P", [63, 64, 65])
def test_schedules_agree_around_the_limit(P):
    """64 x 64 pixels: 64 points are 4096 waves."""
    gs, pts = system(64, 64, 2)
    out = []
    for ppt, block in ((1, 128), (1, 256), (1, 512), (2, 256)):
        ctx = context_with(ppt, block)
        out.append(lensed.loglike_batch(pts[:P].contiguous(), np.zeros(P, np.int32), [gs], ctx=ctx).cpu())
        assert ctx.batch_schedule()["render_block"] == block
        ctx.close()
    assert all(torch.equal(out[0], o) for o in out[1:])
