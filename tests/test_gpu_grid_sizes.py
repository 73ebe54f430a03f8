"""Gradient and residual of gridded functions on the smallest grids and on ones
of a little more points than the launch has threads, against the oracle's
differences: the gradient to 1e-15 and the residual to 1e-9 of the largest
value, as in FP64 elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import grid as G  # noqa: E402
from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("n", [(4, 4), (4, 67), (513, 512), (512, 513), (4, 4, 4), (5, 4, 300), (65, 64, 66)])
def test_grid_sizes(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ctx = pdd.Context(0)
    D = len(n)
    pd = W.unit_square_problem(seed=0) if D == 2 else W.random_problem(np.random.default_rng(3), 3)
    prob = pdd.Problem(ctx, pd)
    lo, hi = W.bounding_box(pd)
    u = np.random.default_rng(sum(n)).normal(size=n[::-1]) * 0.1 + 1.0
    g = {"dim": D, "n": list(n), "lo": lo, "hi": hi, "data": u}
    t = torch.as_tensor(u).cuda().contiguous()
    _, r = pdd.grid_residual(prob, g, t)
    _, outs = pdd.grid_gradient(ctx, g, t)
    r, outs = r.cpu().numpy(), [o.cpu().numpy() for o in outs]
    prob.close()
    ctx.close()
    want = G.residual(pd, g)
    assert np.max(np.abs(r - want)) <= 1e-9 * np.max(np.abs(want))
    ref = G.gradient(g)
    scale = max(np.max(np.abs(x["data"])) for x in ref)
    for got, x in zip(outs, ref):
        assert np.max(np.abs(got - x["data"])) <= 1e-15 * scale
