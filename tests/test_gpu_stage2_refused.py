"""A second-stage call refused for a singular interpolation system (two nodes at
the same point of an interface) leaves u's interior as it was, whichever way its
subdomains would be solved, and the next call is as ever."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("n", [33, 129, 257])
@pytest.mark.parametrize("way", ["cyclic reduction", "substitution", "columns"])
def test_interior_is_left_alone(n, way, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pd = W.unit_square_problem(seed=0)
    if way == "columns":
        pd = dict(pd, c_a=3.0, c_b=0.0)
    if way == "substitution":
        monkeypatch.setenv("PDD_STAGE2_SUBSTITUTE", "1")
    part, nodes = W.unit_square_partition(n), W.unit_square_nodes()
    vals = W.manufactured_u(pd, nodes)
    bad, bad_vals = np.vstack([nodes, nodes[-1:]]), np.append(vals, vals[-1])  # on the last line only
    ctx = pdd.Context(0)
    prob = pdd.Problem(ctx, pd)
    for kept in (False, True):
        u = torch.full((n, n), -7.5, dtype=torch.float64, device="cuda")
        with pytest.raises(pdd.PDDError) as e:
            pdd.stage2(prob, part["n"], part["cuts"], bad, bad_vals, part["rbf_eps"], out=u)
        assert e.value.status == -1 and "0.75" in str(e.value)
        assert bool(torch.all(u[1:-1, 1:-1] == -7.5))
        got = pdd.stage2(prob, part["n"], part["cuts"], nodes, vals, part["rbf_eps"]).cpu().numpy()
        fresh = pdd.Context(0)
        p = pdd.Problem(fresh, pd)
        want = pdd.stage2(p, part["n"], part["cuts"], nodes, vals, part["rbf_eps"]).cpu().numpy()
        p.close()
        fresh.close()
        assert got.tobytes() == want.tobytes()
    prob.close()
    ctx.close()
