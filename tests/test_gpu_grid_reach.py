"""Residual on a grid that reaches far outside the problem's box: the source's
trig arguments are then beyond what they are inside the box. Wave numbers are
whole and points whole or half numbers, so the arguments are exact and the
expected source is that of numpy's sine, to 16 roundings."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402


# 2^27 rad a unit: 2.1e7 revolutions over the box (at most 2^25), 1.4e9 and
# 1.0e10 rad over the grids of 10 and 80 units
@pytest.mark.parametrize("lo,hi", [(0, 1), (0, 10), (0, 80), (-80, 0), (-40, 40)])
@pytest.mark.parametrize("dim,tab", [(2, False), (2, True), (3, False)])
def test_residual_outside_the_box(lo, hi, dim, tab):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    k, n = 2.0 ** 27, 2 * (hi - lo) + 1 if hi - lo > 1 else 5
    pd = {"dim": dim, "domain": "box", "lo": [0.0] * dim, "hi": [1.0] * dim, "sigma": 1.0, "b0": [0.0] * dim,
          "B": [[0.0] * dim] * dim, "c_a": 0.0, "c_b": 0.0, "mono": [], "fx": [], "gx": [], "seed": 0,
          "trig": [{"amp": 1.0, "k": [k + 4.0 * d for d in range(dim)], "phase": [0.5] * dim}]}
    g = {"dim": dim, "n": [n] * dim, "lo": [float(lo)] * dim, "hi": [float(hi)] * dim}
    if tab:  # a tabulated coefficient: the general kernel
        pd["tab"] = {"c": {"dim": dim, "n": [2] * dim, "lo": [-100.0] * dim, "hi": [100.0] * dim,
                           "data": np.zeros([2] * dim)}}
    ctx = pdd.Context(0)
    prob = pdd.Problem(ctx, pd)
    _, r = pdd.grid_residual(prob, g, torch.zeros([n] * dim, dtype=torch.float64, device="cuda"))
    r = r.cpu().numpy()
    prob.close()
    ctx.close()
    x = np.linspace(lo, hi, n)
    s = [np.sin((k + 4.0 * d) * x + 0.5) for d in range(dim)]
    prod = s[1][:, None] * s[0][None, :]
    if dim == 3:
        prod = s[2][:, None, None] * prod[None]
    amp = 0.5 * sum((k + 4.0 * d) ** 2 for d in range(dim))
    assert np.max(np.abs(r + amp * prod)) <= 16 * np.finfo(float).eps * amp
