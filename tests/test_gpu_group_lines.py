"""FP64 walks with a tabulated drift go one path per lane from fewer paths on
than the others: launches on both sides of that line, with and without a buffer
for the hand-over, give the same records bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402


def grid(pd, n, fn):
    lo, hi = W.bounding_box(pd)
    ax = [np.linspace(a, b, n) for a, b in zip(lo, hi)]
    mesh = np.meshgrid(*ax[::-1], indexing="ij")[::-1]
    return {"dim": len(lo), "n": [n] * len(lo), "lo": list(lo), "hi": list(hi), "data": fn(*mesh)}


@pytest.mark.parametrize("dim,below,above", [(2, 65_536, 65_537), (3, 65_536, 65_537), (2, 200_000, 200_001),
                                             (3, 100_000, 100_001)])
@pytest.mark.parametrize("fused", [True, False])
def test_both_sides(dim, below, above, fused):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pd = dict(W.random_problem(np.random.default_rng(dim), dim))
    pd["tab"] = {"b": [grid(pd, 17 if fused else 16 - d, lambda *x, d=d: 0.3 * x[d]) for d in range(dim)],
                 "c": grid(pd, 17, lambda *x: -1.0 - sum(v * v for v in x)),
                 "f": grid(pd, 17, lambda *x: np.sin(x[0]))}
    nodes = W.face_nodes(np.random.default_rng(1), pd, 1)
    ctx = pdd.Context(0)
    prob = pdd.Problem(ctx, pd)
    opts = dict(dt=1e-2, precision="fp64", stream_id=3)
    got = []
    for n in (below, above):
        for noalloc in (False, True):
            rec = pdd.alloc_records(n)
            kw = dict(opts, n_paths=n, records=rec)
            out = pdd.alloc_stats(1)
            if noalloc:
                pdd.solve_nodes_noalloc(prob, nodes, out, **kw)
            else:
                pdd.solve_nodes(prob, nodes, out=out, **kw)
            torch.cuda.synchronize()
            got.append([rec[k].cpu().numpy()[:below] for k in ("phi", "steps")])
    for g in got[1:]:
        for a, b in zip(g, got[0]):
            np.testing.assert_array_equal(a, b)
    prob.close()
    ctx.close()
