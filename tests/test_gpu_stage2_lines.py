"""The interface lines of the second stage against the oracle: as many data
points as one wave solves for and one more, lines next to each other and to the
box's edge (subdomains without interior points, or none with any), lines that
cross, cuts in no order. And a refused call in their company: one line of
several singular."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import stage2 as S2  # noqa: E402
from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("n,cuts,count", [
    ((3, 3), [[0.5], []], 1), ((3, 5), [[], [0.5, 0.25]], 2), ((5, 5), [[0.25, 0.5, 0.75], [0.5]], 3),
    ((9, 17), [[0.5, 0.25], [0.75, 0.5]], 5), ((33, 65), [[0.75, 0.25, 0.5], [0.5, 0.53125]], 13),
    ((65, 33), [[0.5], [0.25]], 14), ((65, 65), [[0.25, 0.5], [0.5]], 15), ((17, 1301), [[0.5], []], 20)])
def test_lines(n, cuts, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pd = W.unit_square_problem(seed=0)
    rng = np.random.default_rng(count)
    t = (np.arange(count) + rng.uniform(0.2, 0.8, count) + 0.5) / (count + 1)
    nodes = np.concatenate([np.column_stack([np.full(count, c), t] if a == 0 else [t, np.full(count, c)])
                            for a in (0, 1) for c in cuts[a]])
    vals = rng.normal(size=len(nodes))
    eps = 2.0 * (count + 1)
    ctx = pdd.Context(0)
    prob = pdd.Problem(ctx, pd)
    ref = S2.stage2(pd, n, cuts, nodes, vals, eps)
    for _ in range(2):
        u = pdd.stage2(prob, n, cuts, nodes, vals, eps).cpu().numpy()
        assert np.max(np.abs(u - ref) / np.maximum(1.0, np.abs(ref))) <= 1e-10
    with pytest.raises(pdd.PDDError) as e:  # the first node of the last line twice
        pdd.stage2(prob, n, cuts, np.vstack([nodes, nodes[-count:][:1]]), np.append(vals, 0.0), eps)
    assert e.value.status == -1
    assert pdd.stage2(prob, n, cuts, nodes, vals, eps).cpu().numpy().tobytes() == u.tobytes()
    prob.close()
    ctx.close()
