"""The second stage's kernels at the edges of their ranges. Block cyclic
reduction: two subdomains of different widths (the blocks are padded to the wider one, a
multiple of 16) over one to 130 block rows, along either axis, against the
oracle's sparse direct solves to the second stage's 1e-10. A repeated call,
which takes the kept factors, gives the same bits. Interpolation weights: lines
with no node, with as many as fit in LDS and with more, and a repeated node."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = pdd.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("w1,w2,rows", [(1, 2, 1), (1, 15, 3), (16, 17, 2), (31, 33, 5), (32, 40, 64), (48, 49, 127),
                                        (63, 64, 130)])
def test_block_edges(ctx, axis, w1, w2, rows):
    from oracle import stage2 as S2
    pd = dict(W.unit_square_problem(seed=0), b0=[3.0, -2.0])
    n = [w1 + w2 + 3, rows + 2]
    cut = (w1 + 1) / (n[0] - 1)
    nodes = np.column_stack([np.full(4, cut), [0.2, 0.4, 0.6, 0.8]])
    cuts = [[cut], []]
    if axis == 1:
        n, nodes, cuts = n[::-1], nodes[:, ::-1].copy(), cuts[::-1]
    vals = W.manufactured_u(pd, nodes) + np.random.default_rng(w1).normal(scale=0.01, size=len(nodes))
    prob = pdd.Problem(ctx, pd)
    got = [pdd.stage2(prob, tuple(n), cuts, nodes, vals, 3.0).cpu().numpy() for _ in range(2)]
    prob.close()
    ref = S2.stage2(pd, tuple(n), cuts, nodes, vals, 3.0)
    assert np.max(np.abs(got[0] - ref) / np.maximum(1.0, np.abs(ref))) <= 1e-10
    assert got[0].tobytes() == got[1].tobytes()


def test_unlike_boxes(ctx):
    """Interfaces on both axes: 10 to 200 points a side, one subdomain with
    fewer block rows than the others' upper levels leave out."""
    from oracle import stage2 as S2
    pd = dict(W.unit_square_problem(seed=0), b0=[3.0, -2.0])
    n = (10 + 60 + 3, 30 + 200 + 3)
    cuts = [[11 / (n[0] - 1)], [31 / (n[1] - 1)]]
    nodes = np.array([[cuts[0][0], y] for y in (0.05, 0.4, 0.8)] + [[x, cuts[1][0]] for x in (0.05, 0.4, 0.8)])
    vals = W.manufactured_u(pd, nodes) + np.random.default_rng(1).normal(scale=0.01, size=len(nodes))
    prob = pdd.Problem(ctx, pd)
    got = [pdd.stage2(prob, n, cuts, nodes, vals, 3.0).cpu().numpy() for _ in range(2)]
    prob.close()
    ref = S2.stage2(pd, n, cuts, nodes, vals, 3.0)
    assert np.max(np.abs(got[0] - ref) / np.maximum(1.0, np.abs(ref))) <= 1e-10
    assert got[0].tobytes() == got[1].tobytes()


@pytest.mark.parametrize("count", [0, 1, 62, 63, 134, 135, 300])
def test_weights(ctx, count):
    from oracle import stage2 as S2
    pd = W.unit_square_problem(seed=0)
    rng = np.random.default_rng(count)
    t = (np.arange(count) + rng.uniform(0.2, 0.8, count) + 0.5) / (count + 1)
    rng.shuffle(t)
    nodes = np.column_stack([np.full(count, 0.5), t]).reshape(count, 2)
    vals = rng.normal(size=count)
    eps, n, cuts = 2.0 * (count + 1), (65, 65), [[0.25, 0.5], []]
    prob = pdd.Problem(ctx, pd)
    u = pdd.stage2(prob, n, cuts, nodes, vals, eps).cpu().numpy()
    ref = S2.stage2(pd, n, cuts, nodes, vals, eps)
    assert np.max(np.abs(u - ref) / np.maximum(1.0, np.abs(ref))) <= 1e-10
    if count:
        with pytest.raises(pdd.PDDError) as e:
            pdd.stage2(prob, n, cuts, np.vstack([nodes, nodes[:1]]), np.append(vals, vals[0]), eps)
        assert e.value.status == -1
    assert pdd.stage2(prob, n, cuts, nodes, vals, eps).cpu().numpy().tobytes() == u.tobytes()
    prob.close()
