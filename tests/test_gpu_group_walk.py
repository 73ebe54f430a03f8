"""Walks by groups of lanes against one path per lane, bit for bit: a launch of
more than 400,000 paths walks one path per lane and hands its longest walks
over, a smaller one is walked by groups from the start. The same paths in
launches of both kinds, from one path to a few more than a wave's groups hold,
must give the same records, and a batch with hand-overs between its items the
same statistics as its items alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402

BIG = 400_001  # paths of the smallest launch that hands over


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = pdd.Context(0)
    yield c
    c.close()


def case(name):
    """(problem dict, nodes, options) of a walk in the kernel that `name` stands for."""
    if name == "ball":
        return W.ball_killing_problem(2, seed=5), np.array([[0.1, 0.2], [-0.5, 0.6], [0.9, 0.0]]), dict(exit="bridge")
    if name == "tabulated":
        return W.paper_example_problem(33, dtype=np.float32, seed=5), W.paper_example_nodes()[::7], dict(exit="bridge")
    if name == "cube":
        pd = W.random_problem(np.random.default_rng(5), 3)
        return pd, W.face_nodes(np.random.default_rng(6), pd, 3), dict(exit="bridge")
    if name == "capped":
        return W.unit_square_problem(5), W.unit_square_nodes()[::7], dict(exit="bridge", max_steps=37)
    return W.unit_square_problem(5), W.unit_square_nodes()[::7], dict(exit=name)


def solve(ctx, prob, pd, nodes, est, n, opts, precision):
    rec = pdd.alloc_records(len(nodes) * n, correction=est != "plain")
    rec["steps"].zero_()
    kw = dict(opts, n_paths=n, precision=precision, records=rec)
    dt = np.float64 if precision == "fp64" else np.float32
    if est == "correction":
        u, r, _ = W.correction_grids(pd, 17, seed=3, dtype=dt)
        g = [torch.as_tensor(x["data"]).cuda() for x in (u, r)]
        pdd.solve_correction(prob, u, g[0], r, g[1], nodes, plain_alongside=True, **kw)
    elif est == "ito":
        gd = W.gradient_grids(pd, 17, seed=3, dtype=dt)
        pdd.solve_ito(prob, gd, [torch.as_tensor(x["data"]).cuda() for x in gd], nodes, **kw)
    else:
        pdd.solve_nodes(prob, nodes, **kw)
    torch.cuda.synchronize()
    return [v.cpu().numpy().reshape(len(nodes), n) for v in rec.values() if v is not None]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("name,est", [("bridge", "plain"), ("bridge", "correction"), ("bridge", "ito"),
                                      ("shift", "plain"), ("naive", "correction"), ("capped", "plain"),
                                      ("ball", "plain"), ("tabulated", "plain"), ("cube", "plain"),
                                      ("cube", "correction"), ("cube", "ito")])
def test_groups_equal_lanes(ctx, name, est, precision):
    pd, nodes, opts = case(name)
    opts = dict(opts, dt=4e-3, stream_id=9)
    prob = pdd.Problem(ctx, pd)
    n = -(-BIG // len(nodes))
    big = solve(ctx, prob, pd, nodes, est, n, opts, precision)
    for k in (1, 2, 3, 5, 17, 64, 300, 30_000):
        part = solve(ctx, prob, pd, nodes, est, k, opts, precision)
        for a, b in zip(part, big):
            np.testing.assert_array_equal(a, b[:, :k])
    # the rest of the big launch's paths, by groups
    half = n // 2
    part = solve(ctx, prob, pd, nodes, est, n - half, dict(opts, path_offset=half), precision)
    for a, b in zip(part, big):
        np.testing.assert_array_equal(a, b[:, half:])
    prob.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dim", [2, 3])
def test_batch_hand_over(ctx, dim, precision):
    """Items of very different sizes and walk lengths, ragged and uniform."""
    rng = np.random.default_rng(dim)
    items = []
    for q, total in enumerate((250_000, 3, 130_000, 1, 20_000, 77)):
        pd = W.random_problem(rng, dim)
        n_nodes = min(total, 7)
        opts = dict(dt=(2e-3, 2e-2)[q % 2], precision=precision, stream_id=q)
        if q % 2:
            opts["n_paths"] = -(-total // n_nodes)
        else:
            counts = rng.multinomial(total - 2 * n_nodes, rng.dirichlet(np.ones(n_nodes))) + 2
            opts["n_paths_per_node"] = counts.astype(np.uint64)
        items.append({"problem": pdd.Problem(ctx, pd), "nodes": W.face_nodes(rng, pd, n_nodes), "opts": opts})
    both = [pdd.stats_to_numpy(o) for o in pdd.solve_batch(ctx, items)]
    for it, b in zip(items, both):
        alone = pdd.stats_to_numpy(pdd.solve_nodes(it["problem"], it["nodes"], **it["opts"]))
        assert alone.tobytes() == b.tobytes()
        it["problem"].close()
