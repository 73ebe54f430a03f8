"""The second stage over the operators that decide how its subdomains are
solved: cell Peclet numbers |b| dx / sigma^2 on both sides of 1, up to 2e5, and
killing rates of either sign, analytic and tabulated. Two subdomains of 63 x 63
unknowns; each is compared with the exact solution of its five-point system
(sparse LU refined in extended precision) for the boundary values that the
call gave it. Allowed is four times the error of banded LU without pivoting in
FP64, computed here, and 16 roundings."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1512_02818_amd import pdd  # noqa: E402
from paper_1512_02818_amd import workloads as W  # noqa: E402

DX, M = 1.0 / 256, 63


def apply(st, x):
    """The five-point operator, coefficients [west, south, centre, north, east] at every point, on an array [y][x]."""
    r = st[2] * x
    r[:, 1:] += st[0][:, 1:] * x[:, :-1]
    r[:, :-1] += st[4][:, :-1] * x[:, 1:]
    r[1:] += st[1][1:] * x[:-1]
    r[:-1] += st[3][:-1] * x[1:]
    return r


def bands(st):
    """Its coefficients in rows of 2 w + 1, in the order of the points."""
    rows, w = st[2].shape
    A = np.zeros((rows, w, 2 * w + 1))
    A[:, :, w], A[1:, :, 0], A[:-1, :, 2 * w] = st[2], st[1][1:], st[3][:-1]
    A[:, 1:, w - 1], A[:, :-1, w + 1] = st[0][:, 1:], st[4][:, :-1]
    return A.reshape(rows * w, 2 * w + 1)


def exact(st, f):
    import scipy.sparse as sp
    import scipy.sparse.linalg as sl
    w, A = f.shape[1], bands(st)
    off = sorted({-w, -1, 0, 1, w})
    lu = sl.splu(sp.diags([A[max(0, -o):len(A) - max(0, o), w + o] for o in off], off, format="csc"))
    x, wide = np.zeros(f.shape, np.longdouble), [v.astype(np.longdouble) for v in st]
    for _ in range(12):
        x = x + lu.solve((f - apply(wide, x)).astype(np.float64).ravel()).reshape(f.shape)
    return x


def banded_lu(st, f):
    w, A = f.shape[1], bands(st)
    n, y, o = len(A), f.astype(np.float64).ravel(), np.arange(w)
    x = np.zeros(n + w)
    for k in range(n - 1):
        m = min(w, n - 1 - k)
        rows = k + 1 + o[:m]
        mult = A[rows, w - 1 - o[:m]] / A[k, w]
        A[rows[:, None], o[None] - o[:m, None] + w] -= mult[:, None] * A[k, w + 1:]
        y[rows] -= mult * y[k]
    for k in range(n - 1, -1, -1):
        x[k] = (y[k] - A[k, w + 1:] @ x[k + 1:k + 1 + w]) / A[k, w]
    return x[:n].reshape(f.shape)


def errors(pd, u, lo, dx, box, b, c):
    """Errors, relative to the largest value, of the values u inside box = (i0, i1, j0, j1) and of banded LU
    (by rows along the shorter side), for u's values on the box's edges; b(x, y), c(x, y): the coefficients."""
    from oracle import oracle as O
    i0, i1, j0, j1 = box
    x, y = np.meshgrid(lo[0] + np.arange(i0 + 1, i1) * dx[0], lo[1] + np.arange(j0 + 1, j1) * dx[1])
    b, c = b(x, y), c(x, y)
    h = [0.5 * pd["sigma"] ** 2 / d ** 2 for d in dx]
    st = [h[0] - b[0] / (2 * dx[0]), h[1] - b[1] / (2 * dx[1]), -2 * h[0] - 2 * h[1] + c + 0 * x,
          h[1] + b[1] / (2 * dx[1]), h[0] + b[0] / (2 * dx[0])]
    f = O.source(pd, np.stack([x.ravel(), y.ravel()], axis=1)).reshape(x.shape).astype(np.longdouble)
    v = u[j0:j1 + 1, i0:i1 + 1].astype(np.longdouble)
    f[:, 0] -= st[0][:, 0] * v[1:-1, 0]
    f[0] -= st[1][0] * v[0, 1:-1]
    f[-1] -= st[3][-1] * v[-1, 1:-1]
    f[:, -1] -= st[4][:, -1] * v[1:-1, -1]
    v = v[1:-1, 1:-1]
    if f.shape[1] > f.shape[0]:
        f, v, st = f.T.copy(), v.T.copy(), [st[q].T.copy() for q in (1, 0, 2, 4, 3)]
    ref = exact(st, f)
    return [float(np.max(np.abs(e - ref)) / np.max(np.abs(ref))) for e in (v, banded_lu(st, f))]


def constant_grid(v):
    return {"dim": 2, "n": [2, 2], "lo": [0.0, 0.0], "hi": [0.5, 0.25], "data": np.full((2, 2), float(v))}


@pytest.mark.parametrize("b,sigma,c,tab", [
    (0.0, 1.0, -1.0, ()), (64.0, 1.0, -1.0, ()), (255.0, 1.0, 0.0, ()), (257.0, 1.0, 0.0, ()), (50.0, 0.1, -1.0, ()),
    (50.0, 0.01, -1.0, ()), (5000.0, 0.01, -1.0, ()), (0.0, 1.0, 40.0, ()), (0.0, 1.0, 150.0, ()),
    (64.0, 1.0, -1.0, "b"), (512.0, 1.0, -1.0, "b"), (64.0, 0.125, -1.0, "bc"), (0.0, 1.0, 150.0, "c")])
def test_operators(b, sigma, c, tab):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    pd = dict(W.unit_square_problem(seed=0), lo=[0.0, 0.0], hi=[0.5, 0.25], sigma=sigma, B=[[0.0, 0.0], [0.0, 0.0]],
              b0=[b, -b], c_a=c, c_b=0.0)
    if tab:
        pd["tab"] = {}
        if "b" in tab:
            pd["tab"]["b"] = [constant_grid(b), constant_grid(-b)]
        if "c" in tab:
            pd["tab"]["c"] = constant_grid(c)
    nodes = np.array([[0.25, y] for y in (0.05, 0.1, 0.15, 0.2)])
    vals = W.manufactured_u(pd, nodes) + np.random.default_rng(1).normal(scale=0.01, size=len(nodes))
    ctx = pdd.Context(0)
    prob = pdd.Problem(ctx, pd)
    got = [pdd.stage2(prob, (2 * M + 3, M + 2), [[0.25], []], nodes, vals, 3.0).cpu().numpy() for _ in range(2)]
    prob.close()
    ctx.close()
    assert got[0].tobytes() == got[1].tobytes()  # the second call takes what the first kept
    for i0 in (0, M + 1):
        err, lu = errors(pd, got[0], (0.0, 0.0), (DX, DX), (i0, i0 + M + 1, 0, M + 1),
                         lambda x, y: (b + 0 * x, -b + 0 * x), lambda x, y: c)
        print(f"b {b} sigma {sigma} c {c} {tab}: {err:.1e}, banded LU {lu:.1e}", flush=True)
        assert err <= 4 * lu + 16 * np.finfo(float).eps


@pytest.mark.parametrize("w,rows", [(1, 7), (15, 15), (16, 255), (31, 127), (33, 63), (47, 191), (63, 63), (64, 255)])
@pytest.mark.parametrize("axis,laplace", [(0, False), (1, False), (0, True)])
def test_strips(w, rows, axis, laplace):
    """Strips of every width of the cyclic reduction's blocks, over one to eight levels, with an operator that
    varies and with the Laplacian, whose rounding errors are alike in all rows: no further from exact than the
    banded LU, but for twice (the errors are maxima of rounding noise)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = [2 * w + 3, rows + 2]
    hi = [(m - 1) * DX for m in n]
    nodes = np.array([[(w + 1) * DX, hi[1] * t] for t in (0.2, 0.4, 0.6, 0.8)])
    cuts = [[(w + 1) * DX], []]
    if axis:
        n, hi, nodes, cuts = n[::-1], hi[::-1], nodes[:, ::-1].copy(), cuts[::-1]
    pd = dict(W.unit_square_problem(seed=0), lo=[0.0, 0.0], hi=hi)
    if laplace:
        pd.update(B=[[0.0, 0.0], [0.0, 0.0]], c_a=0.0, c_b=0.0)
    vals = W.manufactured_u(pd, nodes) + np.random.default_rng(w).normal(scale=0.01, size=len(nodes))
    ctx = pdd.Context(0)
    prob = pdd.Problem(ctx, pd)
    u = pdd.stage2(prob, tuple(n), cuts, nodes, vals, 3.0).cpu().numpy()
    prob.close()
    ctx.close()
    B = pd["B"]
    for s0 in (0, w + 1):
        box = (s0, s0 + w + 1, 0, rows + 1)
        err, lu = errors(pd, u, (0.0, 0.0), (DX, DX), box[2:] + box[:2] if axis else box,
                         lambda x, y: (B[0][0] * x, B[1][1] * y), lambda x, y: pd["c_a"] + pd["c_b"] * (x * x + y * y))
        print(f"{w} x {rows}, axis {axis}, {laplace}: {err:.1e}, banded LU {lu:.1e}", flush=True)
        assert err <= 2 * lu + 4 * np.finfo(float).eps


def test_sizes_apart():
    """Strips of 63 columns and of 1, 5, 17 and 40 beside each other, 511 rows: 2.1 GB with blocks of one size, so
    each of the four sizes (16, 32, 48, 64) has its own."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    widths = [1, 63, 5, 1, 40, 17] + [1] * 12
    edges = np.cumsum([0] + [w + 1 for w in widths])
    rows, lines = 511, edges[1:-1]
    n = (int(edges[-1]) + 1, rows + 2)
    pd = dict(W.unit_square_problem(seed=0), lo=[0.0, 0.0], hi=[(m - 1) * DX for m in n])
    nodes = np.array([[i * DX, y] for i in lines for y in (0.4, 1.1, 1.7)])
    vals = W.manufactured_u(pd, nodes) + np.random.default_rng(2).normal(scale=0.01, size=len(nodes))
    ctx = pdd.Context(0)
    prob = pdd.Problem(ctx, pd)
    got = [pdd.stage2(prob, n, [[i * DX for i in lines], []], nodes, vals, 3.0).cpu().numpy() for _ in range(2)]
    prob.close()
    ctx.close()
    assert got[0].tobytes() == got[1].tobytes()
    B = pd["B"]
    for q in (0, 1, 2, 4, 5, 6, 17):
        err, lu = errors(pd, got[0], (0.0, 0.0), (DX, DX), (int(edges[q]), int(edges[q + 1]), 0, rows + 1),
                         lambda x, y: (B[0][0] * x, B[1][1] * y), lambda x, y: pd["c_a"] + pd["c_b"] * (x * x + y * y))
        print(f"width {widths[q]}: {err:.1e}, banded LU {lu:.1e}", flush=True)
        assert err <= 2 * lu + 4 * np.finfo(float).eps
