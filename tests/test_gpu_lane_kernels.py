"""The kernels that walk one path per lane, which only launches of more than
400,000 paths reach, under every launch shape: block, grab, refill period, form
of the bridge test, several launches, hand-over regions that fill up. Their
records are those of the group walk (the same paths in launches below that
line), bit for bit; statistics those of the items alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402

PER_NODE = 133_334  # three nodes: 400,002 paths
# block, workgroups per CU, grab, paths per launch, refill
SHAPES = [(64, 0, 16, 0, 1), (128, 0, 256, 0, 8), (256, 1, 4096, 0, 4), (256, 0, 64, 400_001, 2)]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = pdd.Context(0)
    yield c
    c.close()


def inputs(dim, est, precision):
    """Problem, nodes (the last one inside the shifted test's band) and a solve of their paths into records."""
    pd = W.unit_square_problem(5) if dim == 2 else W.random_problem(np.random.default_rng(5), 3)
    lo, hi = W.bounding_box(pd)
    at = [[0.3, 0.6, 0.4], [0.5, 0.2, 0.7], [1e-3, 0.5, 0.5]]
    nodes = np.array([[a + t * (b - a) for a, b, t in zip(lo, hi, x)] for x in at])
    dt = np.float64 if precision == "fp64" else np.float32
    grids = W.correction_grids(pd, 17, seed=3, dtype=dt)[:2] if est == "correction" else \
        W.gradient_grids(pd, 17, seed=3, dtype=dt) if est == "ito" else []
    tensors = [torch.as_tensor(g["data"]).cuda() for g in grids]

    def solve(prob, n, **opts):
        rec = pdd.alloc_records(len(nodes) * n, correction=est != "plain")
        kw = dict(dt=4e-3, stream_id=9, n_paths=n, precision=precision, records=rec, max_steps=150, **opts)
        if est == "correction":
            pdd.solve_correction(prob, grids[0], tensors[0], grids[1], tensors[1], nodes, plain_alongside=True, **kw)
        elif est == "ito":
            pdd.solve_ito(prob, grids, tensors, nodes, **kw)
        else:
            pdd.solve_nodes(prob, nodes, **kw)
        torch.cuda.synchronize()
        return [rec[k].cpu().numpy().reshape(len(nodes), n) for k in ("steps", "phi", "e") if rec[k] is not None]

    return pd, solve


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("est", ["plain", "correction", "ito"])
@pytest.mark.parametrize("kernel", ["sparse", "dense", "shift", "naive"])
def test_launch_shapes(ctx, kernel, est, dim, precision):
    pd, solve = inputs(dim, est, precision)
    prob = pdd.Problem(ctx, pd)
    opts = {"exit": kernel if kernel in ("shift", "naive") else "bridge"}
    bridge = {"sparse": 1, "dense": 2}.get(kernel, 0)
    half = PER_NODE // 2
    want = [np.concatenate(v, axis=1) for v in zip(solve(prob, half, **opts), solve(prob, half, path_offset=half, **opts))]
    for shape in SHAPES:
        got = solve(prob, PER_NODE, tuning=shape + (bridge,), **opts)
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
    prob.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("est", ["plain", "correction"])
def test_launches_that_each_hand_over(ctx, est, precision):
    """Three launches of 410,000 paths, each with a hand-over, and a smaller one, cut within nodes."""
    pd, solve = inputs(2, est, precision)
    prob = pdd.Problem(ctx, pd)
    n, parts = 440_000, 4
    pieces = [solve(prob, n // parts, path_offset=q * (n // parts), exit="bridge") for q in range(parts)]
    want = [np.concatenate(v, axis=1) for v in zip(*pieces)]
    got = solve(prob, n, exit="bridge", tuning=(256, 0, 64, 410_000))
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)
    prob.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dim", [2, 3])
def test_full_hand_over_regions(ctx, dim, precision):
    """40 items of very short walks beside one of long walks. The items share
    2^19 hand-over entries, in proportion to what their waves may ask for, so the
    long one has some 12,800; the launch's waves, some thousands, all end up with
    it, with up to 16 paths left each."""
    rng = np.random.default_rng(dim)
    pd = W.random_problem(rng, dim)
    prob = pdd.Problem(ctx, pd)
    nodes = W.face_nodes(rng, pd, 2)
    items = [{"problem": prob, "nodes": nodes, "opts": dict(dt=1e-3 * (1 + 1e-3 * q), n_paths=50_000, max_steps=8,
                                                            precision=precision, stream_id=q)} for q in range(40)]
    items.insert(20, {"problem": prob, "nodes": nodes, "opts": dict(dt=2e-3, n_paths=300_000, precision=precision)})
    both = [pdd.stats_to_numpy(o) for o in pdd.solve_batch(ctx, items)]
    for it, b in zip(items, both):
        alone = pdd.stats_to_numpy(pdd.solve_nodes(it["problem"], it["nodes"], **it["opts"]))
        assert alone.tobytes() == b.tobytes()
    prob.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_many_small_items(ctx, precision):
    """1,500 items of 300 paths, ragged and uniform, in any launch shape."""
    rng = np.random.default_rng(7)
    probs = []
    items = []
    for q in range(1500):
        if q % 100 == 0:
            pd = W.random_problem(rng, 2)
            probs.append(pdd.Problem(ctx, pd))
        nodes = W.face_nodes(rng, pd, 3)
        opts = dict(dt=5e-3, precision=precision, stream_id=q, max_steps=100 + q % 7)
        if q % 2:
            opts["n_paths"] = 100
        else:
            opts["n_paths_per_node"] = np.array([1 + q % 50, 200, 99 - q % 50], dtype=np.uint64)
        items.append({"problem": probs[-1], "nodes": nodes, "opts": opts})
    base = torch.cat(pdd.solve_batch(ctx, items)).cpu().numpy()
    for shape in SHAPES[:3]:
        for it in items:
            it["opts"]["tuning"] = shape
        got = torch.cat(pdd.solve_batch(ctx, items)).cpu().numpy()
        assert got.tobytes() == base.tobytes()
    for q in (0, 1, 700, 1499):  # groups, each item alone
        it = items[q]
        alone = pdd.solve_nodes(it["problem"], it["nodes"], **it["opts"]).cpu().numpy()
        lo = 3 * q * pdd.STATS_DTYPE.itemsize
        assert alone.tobytes() == base.tobytes()[lo:lo + alone.nbytes]
    for p in probs:
        p.close()
