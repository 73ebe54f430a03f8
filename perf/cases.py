"""The work that users of this library have it do, as a list of timed calls
through its public entry points: plain, correction and Ito solves of both
precisions from a few thousand paths to many millions, uneven batches, solves
to a tolerance, served requests, the second stage, and the grid operators of
the outer iteration.

`listed()` gives the named cases, `draw(rng)` another case of the same ranges,
`prepare(case, seed)` the state that a program has in hand before the call,
`run(state)` one call, `work(case)` the bytes and arithmetic operations that
one call cannot do without, and `exact(case, seed)` the call's outputs in 64
bits by plain torch and numpy (None where that takes too long).
"""
import math

import numpy as np
import torch

from paper_1512_02818_amd import pdd, tuning
from paper_1512_02818_amd import workloads as W

_shared = {}


def _context():
    """One context for the process, with the tuned launch shapes, as a program keeps it."""
    if "ctx" not in _shared:
        _shared["ctx"] = pdd.Context(0)
        tuning.load(_shared["ctx"])
    return _shared["ctx"]


# --------------------------------------------------------------------------- cases
def listed():
    return [
        # The paper's first-stage solve in double precision: unit square, 18 interface nodes.
        dict(name="plain64_unit", kind="solve", est="plain", precision="fp64", problem="unit", nodes=18,
             paths=10_000, dt=1e-3, exit="bridge"),
        # The same solve at the step that an RMS error of 1e-3 takes: what control variates are compared with.
        dict(name="plain64_unit_fine", kind="solve", est="plain", precision="fp64", problem="unit", nodes=18,
             paths=20_000, dt=1e-4, exit="bridge"),
        # Throughput: long walks from every interface node of the 8 x 8 partition of [0, 4]^2.
        dict(name="plain32_square4", kind="solve", est="plain", precision="fp32", problem="square4", nodes=1792,
             paths=8192, dt=1e-4, exit="bridge"),
        # First iterate of the multigrid-like iteration: few paths, where latency counts.
        dict(name="corr32_unit_small", kind="solve", est="correction", precision="fp32", problem="unit", nodes=18,
             paths=1000, dt=1e-3, exit="bridge", grid=257),
        # Its last iterate, with the plain score beside it for the variance reduction.
        dict(name="corr32_unit_large", kind="solve", est="correction", precision="fp32", problem="unit", nodes=18,
             paths=100_000, dt=1e-3, exit="bridge", grid=257, alongside=True),
        # A 3D correction solve: many nodes of a random cube, an odd path count.
        dict(name="corr32_cube", kind="solve", est="correction", precision="fp32", problem="random3", nodes=333,
             paths=1501, dt=1e-3, exit="bridge", grid=65),
        # Tabulated coefficients, source and boundary data: the paper's own example on 513^2 grids.
        dict(name="plain32_tabulated", kind="solve", est="plain", precision="fp32", problem="paper", nodes=18,
             paths=100_000, dt=1e-3, exit="bridge", grid=513),
        # Many small uneven problems in one call, 2D and 3D together.
        dict(name="batch32_uneven", kind="batch", problems=64, nodes_hi=5000, scale=1e-3),
        # One level of the outer iteration: per-node steps and path counts to a standard error, Ito control variate.
        dict(name="level_ito", kind="level", problem="unit", accuracy=5e-3, pilot=128, grid=129),
        # Served requests of different sizes and tolerances arriving together.
        dict(name="serve_burst", kind="serve", requests=16, nodes_hi=200, tol=1e-2),
        # The second stage when the operator has changed since the last call (a coefficient iteration).
        dict(name="stage2_new_operator", kind="stage2", problem="unit", grid=257),
        # Gradient and residual of a gridded approximation, once per level of the outer iteration.
        dict(name="grids64", kind="grids", dim=2, precision="fp64", n0=513, n1=513),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_solve(rng):
    est = rng.choice(["plain", "plain", "correction", "ito"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    problem = rng.choice(["unit", "square4", "random2", "random3", "ball2"] + (["paper"] if est == "plain" else []))
    if est != "plain" and problem == "ball2":
        problem = "random2"
    dt = rng.choice([1e-3, 5e-4, 2.5e-4] + ([1e-4] if problem in ("unit", "square4") else []))
    nodes = int(_log(rng, 1, 2000))
    # path-steps of the call, at most those of the listed throughput case
    steps = _log(rng, 2e6, 2e10 if prec == "fp32" else 3e9)
    per_path = {"unit": 0.1, "square4": 0.8, "random2": 0.4, "random3": 0.3, "paper": 0.22, "ball2": 0.3}[problem] / dt
    paths = max(2, min(1_000_000, int(steps / per_path / nodes)))
    c = dict(kind="solve", est=est, precision=prec, problem=problem, nodes=nodes, paths=paths, dt=dt,
             exit=rng.choice(["bridge", "bridge", "bridge", "shift"]))
    if est != "plain":
        c["grid"] = rng.choice([129, 257, 513]) if problem != "random3" else rng.choice([33, 65])
        c["alongside"] = est == "correction" and rng.random() < 0.3
    if problem == "paper":
        c["grid"] = rng.choice([129, 257, 513])
    return c


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["batch", "level", "serve", "stage2", "grids"])
    if kind == "solve":
        return _draw_solve(rng)
    if kind == "batch":
        n = int(_log(rng, 3, 64))
        return dict(kind="batch", problems=n, nodes_hi=int(_log(rng, 20, 5000)), scale=_log(rng, 2e-4, 1e-3))
    if kind == "level":
        return dict(kind="level", problem="unit", accuracy=_log(rng, 3e-3, 0.1), pilot=rng.choice([64, 128, 500]),
                    grid=rng.choice([65, 129, 257]))
    if kind == "serve":
        return dict(kind="serve", requests=rng.randint(2, 16), nodes_hi=int(_log(rng, 5, 200)), tol=1e-2)
    if kind == "stage2":
        if rng.random() < 0.5:
            return dict(kind="stage2", problem="unit", grid=4 * rng.randint(8, 64) + 1)
        return dict(kind="stage2", problem="square4", grid=8 * rng.randint(8, 48) + 1)
    dim = rng.choice([2, 2, 3])
    lo, hi = (33, 2049) if dim == 2 else (17, 129)
    c = dict(kind="grids", dim=dim, precision=rng.choice(["fp32", "fp64"]), n0=int(_log(rng, lo, hi)),
             n1=int(_log(rng, lo, hi)))
    if dim == 3:
        c["n2"] = int(_log(rng, lo, hi))
    return c


# --------------------------------------------------------------------------- inputs
def _problem(case, seed):
    """The problem dict of a case."""
    kind = case["problem"]
    if kind == "unit":
        return W.unit_square_problem(seed)
    if kind == "square4":
        return W.big_square_problem(seed)
    if kind == "paper":
        return W.paper_example_problem(case["grid"], dtype=np.float32, seed=seed)
    if kind == "ball2":
        return W.ball_killing_problem(2, radius=1.0, c=-1.0, seed=seed)
    dim = 2 if kind == "random2" else 3
    pd = W.random_problem(np.random.default_rng(seed), dim)
    # the side is the case's, not the seed's, so that every seed has as much to do
    side = 2.0
    old = pd["hi"][0]
    pd["hi"] = [side] * dim
    for t in pd["trig"]:
        t["k"] = [k * old / side for k in t["k"]]
    return pd


def _nodes(case, pd, seed):
    n, kind = case["nodes"], case["problem"]
    if kind in ("unit", "paper") and n == 18:
        return W.unit_square_nodes() if kind == "unit" else W.paper_example_nodes()
    if kind == "square4" and n == 1792:
        return W.big_square_nodes()
    rng = np.random.default_rng(seed + 77)
    if kind == "ball2":
        r, th = 0.9 * np.sqrt(rng.uniform(0, 1, n)), rng.uniform(0, 2 * np.pi, n)
        return np.stack([r * np.cos(th), r * np.sin(th)], axis=1)
    return W.face_nodes(rng, pd, n)


def _dtype(precision):
    return np.float64 if precision == "fp64" else np.float32


def _on_gpu(grid):
    return torch.as_tensor(np.ascontiguousarray(grid["data"])).cuda()


def _solve_args(case, pd, seed):
    """Options of a solve and, by estimator, its grids."""
    opts = dict(dt=case["dt"], n_paths=case["paths"], precision=case["precision"], exit=case["exit"])
    dt = _dtype(case["precision"])
    if case["est"] == "correction":
        u, r, _ = W.correction_grids(pd, case["grid"], seed=seed + 1, dtype=dt)
        opts["plain_alongside"] = bool(case.get("alongside"))
        return opts, [u, r]
    if case["est"] == "ito":
        return opts, W.gradient_grids(pd, case["grid"], seed=seed + 1, dtype=dt)
    return opts, []


def _stage2_inputs(case, seed):
    """A problem with an operator of its own for each seed, its partition, nodes and nodal values."""
    rng = np.random.default_rng(seed)
    pd = _problem(case, seed)
    pd["c_a"] = -float(rng.uniform(0.5, 1.5))
    pd["B"] = [[float(rng.uniform(-0.5, 0.5)), 0.0], [0.0, float(rng.uniform(-0.5, 0.5))]]
    if case["problem"] == "unit":
        part, nodes = W.unit_square_partition(case["grid"]), W.unit_square_nodes()
    else:
        part, nodes = W.big_square_partition(case["grid"]), W.big_square_nodes()
    values = W.manufactured_u(pd, nodes) + 1e-3 * rng.standard_normal(len(nodes))
    return pd, part, nodes, values


def _grids_input(case, seed):
    """A smooth function with some noise, the values that an assembled approximation has."""
    n = [case["n0"], case["n1"]] + ([case["n2"]] if case["dim"] == 3 else [])
    pd = dict(W.random_problem(np.random.default_rng(seed), case["dim"]))
    ax = [torch.linspace(pd["lo"][d], pd["hi"][d], n[d], dtype=torch.float64, device="cuda") for d in range(len(n))]
    u = torch.zeros(n[::-1], dtype=torch.float64, device="cuda")
    for t in pd["trig"]:
        s = [torch.sin(t["k"][d] * ax[d] + t["phase"][d]) for d in range(len(n))]
        v = s[1][:, None] * s[0][None, :]
        u += t["amp"] * (v if len(n) == 2 else s[2][:, None, None] * v[None])
    g = torch.Generator(device="cuda").manual_seed(seed)
    u += 1e-6 * torch.randn(u.shape, dtype=torch.float64, device="cuda", generator=g)
    u = u.to(torch.float64 if case["precision"] == "fp64" else torch.float32).contiguous()
    return pd, {"dim": len(n), "n": n, "lo": list(pd["lo"]), "hi": list(pd["hi"])}, u


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "solve":
        pd = _problem(case, seed)
        s["nodes"] = _nodes(case, pd, seed)
        s["opts"], grids = _solve_args(case, pd, seed)
        s["est"], s["grids"], s["tensors"] = case["est"], grids, [_on_gpu(g) for g in grids]
        s["problem"] = pdd.Problem(_context(), pd)
    elif kind == "batch":
        ctx = _context()
        # the shape of the mix is the case's; the coefficients' random numbers and the paths' are the seed's
        items = W.batch_workload(seed=4, n_problems=case["problems"], node_range=(10, case["nodes_hi"]),
                                 scale=case["scale"])
        s["items"] = []
        for q, it in enumerate(items):
            it["problem"]["seed"] = seed * 1000 + q
            s["items"].append({"problem": pdd.Problem(ctx, it["problem"]), "nodes": it["nodes"],
                               "opts": dict(dt=it["dt"], n_paths=max(2, it["n_paths"]), precision="fp32")})
    elif kind == "level":
        pd = _problem(case, seed)
        nodes = W.unit_square_nodes()
        grad = W.gradient_grids(pd, case["grid"], seed=seed + 1)
        grad_t = [_on_gpu(g) for g in grad]
        prob = pdd.Problem(_context(), pd)
        # each node has its own step, from the bias constant that the fit gave it
        beta = np.random.default_rng(seed).uniform(1.0, 4.0, len(nodes))
        h = np.clip(case["accuracy"] / (2.0 * beta), 1e-5, 1e-2)
        s["items"] = [{"problem": prob, "nodes": nodes[i:i + 1], "grad": grad, "grad_t": grad_t,
                       "opts": dict(dt=float(h[i]), precision="fp32", stream_id=i)} for i in range(len(nodes))]
        s["target"], s["pilot"] = case["accuracy"] / 4.0, case["pilot"]
    elif kind == "serve":
        # a server is its context's only user
        ctx = pdd.Context(0)
        tuning.load(ctx)
        s["server"] = pdd.Server(ctx, epoch_paths=1 << 24)
        # the mix is the case's, the paths are the seed's
        problems, reqs = W.serving_stream(seed=5, rate=case["requests"] * 2.0, duration=4.0, n_problems=6,
                                          node_range=(1, case["nodes_hi"]), tols=(case["tol"],), grid_sizes_2d=(129,),
                                          grid_3d=33)
        for q, pd in enumerate(problems):
            pd["seed"] = seed * 1000 + q
        probs = [pdd.Problem(ctx, pd) for pd in problems]
        s["requests"] = []
        for r in reqs[:case["requests"]]:
            a = dict(problem=probs[r["problem"]], nodes=r["nodes"], dt=r["dt"], target_se=r["target_se"],
                     stream_id=r["stream_id"])
            if r["cv"]:
                u, rs, _ = W.correction_grids(problems[r["problem"]], r["grid_n"], seed=seed + 1)
                a.update(u_prev=u, u_prev_t=_on_gpu(u), resid=rs, resid_t=_on_gpu(rs))
            s["requests"].append(a)
    elif kind == "stage2":
        pd, s["part"], s["nodes"], s["values"] = _stage2_inputs(case, seed)
        s["problem"] = pdd.Problem(_context(), pd)
    else:
        pd, s["grid"], s["u"] = _grids_input(case, seed)
        s["ctx"], s["problem"] = _context(), pdd.Problem(_context(), pd)
    return s


# --------------------------------------------------------------------------- one pass
_FIELDS = ("mean", "var", "stderr", "mean_steps", "mean_plain", "var_plain", "cov", "rho", "vr", "vr_opt")


def _stats(raw):
    """Every field of a solve's statistics (a device buffer of 184-byte records)."""
    n = raw.numel() // pdd.STATS_DTYPE.itemsize
    f = raw.view(torch.float64).view(n, -1)
    out = {"counts": raw.view(torch.int64).view(n, -1)[:, :3], "sums": f[:, 13:]}
    out.update({name: f[:, 3 + k] for k, name in enumerate(_FIELDS)})
    return out


def run(state):
    kind = state["kind"]
    if kind == "solve":
        p, nodes, g, t = state["problem"], state["nodes"], state["grids"], state["tensors"]
        if state["est"] == "correction":
            return _stats(pdd.solve_correction(p, g[0], t[0], g[1], t[1], nodes, **state["opts"]))
        if state["est"] == "ito":
            return _stats(pdd.solve_ito(p, g, t, nodes, **state["opts"]))
        return _stats(pdd.solve_nodes(p, nodes, **state["opts"]))
    if kind == "batch":
        outs = pdd.solve_batch(_context(), state["items"])
        return _stats(torch.cat(outs))
    if kind == "level":
        outs = pdd.solve_to_tolerance(_context(), state["items"], state["target"], state["pilot"], 1 << 30)
        return _stats(torch.cat(outs))
    if kind == "serve":
        server = state["server"]
        ids = [server.submit(**r) for r in state["requests"]]
        if not server.wait_all():
            raise RuntimeError("requests did not complete")
        done = [server.results.pop(i)["stats"] for i in ids]
        all_nodes = np.concatenate(done)
        return {"counts": np.stack([all_nodes[k] for k in ("n", "n_capped", "steps_sum")], axis=1),
                "sums": all_nodes["sums"], **{k: all_nodes[k] for k in _FIELDS}}
    if kind == "stage2":
        part = state["part"]
        return pdd.stage2(state["problem"], part["n"], part["cuts"], state["nodes"], state["values"], part["rbf_eps"])
    _, grad = pdd.grid_gradient(state["ctx"], state["grid"], state["u"])
    _, resid = pdd.grid_residual(state["problem"], state["grid"], state["u"])
    return {"grad": grad, "resid": resid}


# --------------------------------------------------------------------------- what a pass cannot do without
def _mean_exit_time(pd, nodes):
    """E[tau] of the driftless walk from each node (the drift of these problems changes it little)."""
    s2 = pd["sigma"] ** 2
    if pd.get("domain", "box") == "ball":
        r2 = np.sum((nodes - np.asarray(pd["center"])[None, :]) ** 2, axis=1)
        return (pd["radius"] ** 2 - r2) / (pd["dim"] * s2)
    L = np.asarray(pd["hi"]) - np.asarray(pd["lo"])
    x = (nodes - np.asarray(pd["lo"])[None, :]) / L
    odd = np.arange(1, 40 if pd["dim"] == 2 else 16, 2)
    out = np.zeros(len(nodes))
    sines = [np.sin(np.pi * np.outer(x[:, d], odd)) for d in range(pd["dim"])]
    for idx in np.ndindex(*([len(odd)] * pd["dim"])):
        k = odd[list(idx)].astype(np.float64)
        lam = 0.5 * s2 * np.sum((np.pi * k / L) ** 2)
        out += np.prod(4.0 / (np.pi * k)) / lam * np.prod([sines[d][:, i] for d, i in enumerate(idx)], axis=0)
    return out


def _step_ops(dim, est, terms):
    """Arithmetic operations of one step: ten Philox rounds (half a block in 2D), Box-Muller, the affine drift,
    killing, the trig terms of the source, the updates and the exit test; an interpolation per gridded field."""
    n = (20 + 12 if dim == 2 else 40 + 20) + dim * (2 * dim + 4) + 14
    n += terms * (6 * dim + 4) if est != "correction" else 0
    return n + {"plain": 0, "correction": 8 * dim, "ito": 10 * dim}[est]


def _solve_work(pd, nodes, paths, dt, est, grid_bytes=0):
    if len(nodes) > 200:
        tau = _mean_exit_time(pd, nodes[:: len(nodes) // 100]).mean() * len(nodes)
    else:
        tau = _mean_exit_time(pd, nodes).sum()
    flops = tau / dt * paths * _step_ops(pd["dim"], est, len(pd.get("trig", [])) or 1)
    return {"bytes": float(len(nodes) * (8 * pd["dim"] + 184) + grid_bytes), "flops": float(flops)}


def work(case):
    kind = case["kind"]
    if kind == "solve":
        pd = _problem(dict(case, grid=3) if case["problem"] == "paper" else case, 0)
        values = 4 if case["precision"] == "fp32" else 8
        per = {"plain": 5 if case["problem"] == "paper" else 0, "correction": 2, "ito": pd["dim"]}[case["est"]]
        return _solve_work(pd, _nodes(case, pd, 0), case["paths"], case["dt"], case["est"],
                           per * values * case.get("grid", 0) ** pd["dim"])
    if kind == "batch":
        ws = [_solve_work(it["problem"], it["nodes"], max(2, it["n_paths"]), it["dt"], "plain")
              for it in W.batch_workload(seed=4, n_problems=case["problems"], node_range=(10, case["nodes_hi"]),
                                         scale=case["scale"])]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    if kind == "level":
        # V[phi + xi] of this control variate at these steps is about 4 h, and a node has at least its pilot's paths
        h = case["accuracy"] / 5.0
        n = max(case["pilot"], 4 * h / (case["accuracy"] / 4.0) ** 2)
        return _solve_work(W.unit_square_problem(), W.unit_square_nodes(), n, h, "ito", 8 * case["grid"] ** 2)
    if kind == "serve":
        problems, reqs = W.serving_stream(seed=5, rate=case["requests"] * 2.0, duration=4.0, n_problems=6,
                                          node_range=(1, case["nodes_hi"]), tols=(case["tol"],), grid_sizes_2d=(129,),
                                          grid_3d=33)
        # a plain request takes about V / SE^2 paths a node (V about 1), one with a control variate its pilot
        ws = [_solve_work(problems[r["problem"]], r["nodes"], 1000 if r["cv"] else 1.0 / r["target_se"] ** 2,
                          r["dt"], "correction" if r["cv"] else "plain") for r in reqs[:case["requests"]]]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    if kind == "stage2":
        # a banded factorisation and substitution of every subdomain
        n = case["grid"]
        cells, across = (4, 1) if case["problem"] == "unit" else (8, 8)
        w, length = (n - 1) // cells - 1, (n - 1) // across - 1
        w, length = min(w, length), max(w, length)
        unknowns = cells * across * w * length
        return {"bytes": 8.0 * n * n, "flops": unknowns * (2.0 * w * w + 4.0 * w)}
    points = case["n0"] * case["n1"] * case.get("n2", 1)
    size = 8 if case["precision"] == "fp64" else 4
    return {"bytes": float(points * size * (2 + 1 + case["dim"])), "flops": float(points * (60 + 8 * 20 * case["dim"]))}


# --------------------------------------------------------------------------- the same in 64 bits, plainly
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    m = 0xFFFFFFFF
    k0, k1 = seed & m, (seed >> 32) & m
    for _ in range(10):
        lo0, hi0 = _mul32(0xD2511F53, c0)
        lo1, hi1 = _mul32(0xCD9E8D57, c2)
        c0, c1, c2, c3 = hi1 ^ c1 ^ k0, lo1, hi0 ^ c3 ^ k1, lo0
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c0, c1, c2, c3


def _mul32(a, x):
    """Low and high words of the 64-bit product of a 32-bit constant and 32-bit words."""
    a0, a1 = a & 0xFFFF, a >> 16
    p0, p1 = x * a0, x * a1
    t = p0 + ((p1 & 0xFFFF) << 16)
    return t & 0xFFFFFFFF, (p1 >> 16) + (t >> 32)


def _unit(w):
    return (w.double() + 0.5) * 2.0 ** -32


def _normals(step, path, node, seed, dim):
    """The normals of a step: in 2D words 0, 1 (even steps) or 2, 3 (odd steps) of a block of two steps."""
    zero = torch.zeros_like(path)
    w = _philox(zero + (step >> 1 if dim == 2 else step), path, node, zero, seed)
    a, b = (w[0], w[1]) if dim == 3 or step % 2 == 0 else (w[2], w[3])
    r, th = torch.sqrt(-2.0 * torch.log(_unit(a))), 2.0 * math.pi * _unit(b)
    n = [r * torch.cos(th), r * torch.sin(th)]
    if dim == 3:
        n.append(torch.sqrt(-2.0 * torch.log(_unit(w[2]))) * torch.cos(2.0 * math.pi * _unit(w[3])))
    return torch.stack(n, dim=1)


def _u_and_derivatives(pd, x):
    """U, grad U and Lap U of the manufactured solution."""
    u = torch.zeros(len(x), dtype=torch.float64, device=x.device)
    lap, grad, D = torch.zeros_like(u), torch.zeros_like(x), pd["dim"]
    for t in pd.get("trig", []):
        s = [torch.sin(t["k"][d] * x[:, d] + t["phase"][d]) for d in range(D)]
        v = t["amp"] * math.prod(s)
        u, lap = u + v, lap - sum(k * k for k in t["k"]) * v
        for d in range(D):
            grad[:, d] += t["amp"] * t["k"][d] * torch.cos(t["k"][d] * x[:, d] + t["phase"][d]) * math.prod(
                s[:d] + s[d + 1:])
    for m in pd.get("mono", []):
        pw = [[x[:, d] ** max(e - k, 0) * math.prod(range(e - k + 1, e + 1)) for k in range(3)]
              for d, e in enumerate(m["e"])]
        pw = [[p[k] if m["e"][d] >= k else torch.zeros_like(u) for k in range(3)] for d, p in enumerate(pw)]
        u = u + m["coef"] * math.prod(p[0] for p in pw)
        for d in range(D):
            rest = math.prod([p[0] for e, p in enumerate(pw) if e != d])
            grad[:, d] += m["coef"] * pw[d][1] * rest
            lap = lap + m["coef"] * pw[d][2] * rest
    return u, grad, lap


def _interpolate(grid, values, x):
    """Bilinear or trilinear interpolation, cell index and weight clamped to the grid."""
    D, n = grid["dim"], grid["n"]
    i, w = [], []
    for d in range(D):
        t = (x[:, d] - grid["lo"][d]) * ((n[d] - 1) / (grid["hi"][d] - grid["lo"][d]))
        c = t.floor().clamp(0, n[d] - 2)
        i.append(c.long())
        w.append((t - c).clamp(0, 1))
    out = 0.0
    for corner in np.ndindex(*([2] * D)):
        flat, weight = 0, 1.0
        for d in reversed(range(D)):
            flat = flat * n[d] + i[d] + corner[d]
        for d in range(D):
            weight = weight * (w[d] if corner[d] else 1.0 - w[d])
        out = out + weight * values[flat]
    return out


def _walk(pd, nodes, paths, dt, est, grids):
    """Scores phi, e and exit steps of every path of a box problem with the bridge exit test."""
    D, dev = pd["dim"], "cuda"
    lo, hi = (torch.tensor(pd[k], dtype=torch.float64, device=dev) for k in ("lo", "hi"))
    n = len(nodes)
    node = torch.arange(n, device=dev).repeat_interleave(paths)
    path = torch.arange(paths, device=dev).repeat(n)
    x = torch.as_tensor(nodes, dtype=torch.float64, device=dev)[node]
    slot = torch.arange(n * paths, device=dev)
    Y, Z, R = torch.ones(n * paths, dtype=torch.float64, device=dev), 0.0, 0.0
    Z, R = torch.zeros_like(Y), torch.zeros_like(Y)
    phi, e, steps = torch.zeros_like(Y), torch.zeros_like(Y), torch.zeros_like(slot)
    b0, B = (torch.tensor(pd[k], dtype=torch.float64, device=dev)[:D] for k in ("b0", "B"))
    tab, sg = pd.get("tab"), pd["sigma"] * math.sqrt(dt)
    flat = [torch.as_tensor(np.asarray(g["data"], dtype=np.float64)).cuda().reshape(-1) for g in grids]
    tv = {k: torch.as_tensor(np.asarray(tab[k]["data"], dtype=np.float64)).cuda().reshape(-1) for k in "cfg"} if tab else {}
    tb = [torch.as_tensor(np.asarray(g["data"], dtype=np.float64)).cuda().reshape(-1) for g in tab["b"]] if tab else []
    step = 0
    while len(x):
        N = _normals(step, path, node, pd["seed"], D)
        if tab:
            b = torch.stack([_interpolate(tab["b"][d], tb[d], x) for d in range(D)], dim=1)
            c, f = _interpolate(tab["c"], tv["c"], x), _interpolate(tab["f"], tv["f"], x)
        else:
            b = b0[None, :] + x @ B.T
            c = pd["c_a"] + pd["c_b"] * (x * x).sum(1)
            u, grad, lap = _u_and_derivatives(pd, x)
            f = 0.5 * pd["sigma"] ** 2 * lap + (b * grad).sum(1) + c * u
        Z = Z - dt * Y * f
        if est == "correction":
            R = R + dt * Y * _interpolate(grids[1], flat[1], x)
        elif est == "ito":
            R = R - Y * sg * sum(_interpolate(grids[d], flat[d], x) * N[:, d] for d in range(D))
        Y = Y + dt * Y * c
        new = x + dt * b + sg * N
        # exit: outside, or by the bridge between two inside points, face by face
        outside = ((new - lo <= 0) | (hi - new <= 0)).any(1)
        arg = torch.stack([v for d in range(D) for v in ((x[:, d] - lo[d]) * (new[:, d] - lo[d]),
                                                          (hi[d] - x[:, d]) * (hi[d] - new[:, d]))], dim=1)
        arg = arg * (2.0 / sg ** 2)
        p = torch.where(arg <= 36 * math.log(2.0), torch.exp(-arg), torch.zeros_like(arg))
        P = torch.zeros_like(Y)
        for q in range(2 * D):
            P = P + p[:, q] * (1.0 - P)
        zero = torch.zeros_like(path)
        U = _unit(_philox(zero + (step >> 2), path, node, zero + 1, pd["seed"])[step & 3])
        crossed = ~outside & (U < P)
        face = p.argmax(1)
        end = torch.minimum(torch.maximum(new, lo), hi)
        for d in range(D):
            end[:, d] = torch.where(crossed & (face == 2 * d), lo[d], torch.where(crossed & (face == 2 * d + 1), hi[d],
                                                                               end[:, d]))
        step += 1
        done = outside | crossed
        if bool(done.any()):
            xt, at = end[done], slot[done]
            g = _interpolate(tab["g"], tv["g"], xt) if tab else _u_and_derivatives(pd, xt)[0]
            phi[at] = g * Y[done] + Z[done]
            if est == "correction":
                e[at] = (g - _interpolate(grids[0], flat[0], xt)) * Y[done] - R[done]
            elif est == "ito":
                e[at] = phi[at] + R[done]
            steps[at] = step
            keep = ~done
            x, Y, Z, R, slot, path, node = new[keep], Y[keep], Z[keep], R[keep], slot[keep], path[keep], node[keep]
        else:
            x = new
    return phi.view(n, paths), e.view(n, paths), steps.view(n, paths)


def _exact_solve(case, seed):
    pd = _problem(case, seed)
    nodes = _nodes(case, pd, seed)
    opts, grids = _solve_args(case, pd, seed)
    N, est = case["paths"], case["est"]
    phi, e, steps = _walk(pd, nodes, N, case["dt"], est, grids)
    scored = phi if est == "plain" else e
    out = {k: torch.full((len(nodes),), float("nan"), dtype=torch.float64, device="cuda") for k in _FIELDS}
    base = 0.0
    if est == "correction":
        base = _interpolate(grids[0], torch.as_tensor(np.asarray(grids[0]["data"], dtype=np.float64)).cuda().reshape(-1),
                            torch.as_tensor(nodes, device="cuda"))
    out["mean"], out["var"] = base + scored.mean(1), scored.var(1)
    out["stderr"], out["mean_steps"] = torch.sqrt(out["var"] / N), steps.double().mean(1)
    if est != "correction" or opts["plain_alongside"]:
        out["mean_plain"], out["var_plain"] = phi.mean(1), phi.var(1)
        if est != "plain":
            xi = e - phi
            out["cov"] = ((phi - phi.mean(1, keepdim=True)) * (xi - xi.mean(1, keepdim=True))).sum(1) / (N - 1)
            out["rho"] = out["cov"] / torch.sqrt(out["var_plain"] * xi.var(1))
            out["vr"], out["vr_opt"] = out["var_plain"] / out["var"], 1.0 / (1.0 - out["rho"] ** 2)
    return {**out, "counts": None, "sums": None}


def _exact_stage2(case, seed):
    """The interface interpolants and every subdomain's five-point system, solved block by block."""
    pd, part, nodes, values = _stage2_inputs(case, seed)
    n, lo, hi = part["n"], pd["lo"], pd["hi"]
    ax = [lo[d] + (hi[d] - lo[d]) * np.arange(n[d]) / (n[d] - 1) for d in range(2)]
    dx = [(hi[d] - lo[d]) / (n[d] - 1) for d in range(2)]
    X, Yc = np.meshgrid(ax[0], ax[1])
    pts = np.stack([X.ravel(), Yc.ravel()], axis=1)
    U, grad, lap = (t.cpu().numpy() for t in _u_and_derivatives(pd, torch.as_tensor(pts)))
    b = np.asarray(pd["b0"])[None, :2] + pts @ np.asarray(pd["B"]).T
    c = pd["c_a"] + pd["c_b"] * (pts ** 2).sum(1)
    f = (0.5 * lap + (b * grad).sum(1) + c * U).reshape(n[1], n[0])
    b, c, U = b.reshape(n[1], n[0], 2), c.reshape(n[1], n[0]), U.reshape(n[1], n[0])
    u = U.copy()
    u[1:-1, 1:-1] = 0.0
    cuts = [sorted(int(round((x - lo[a]) / dx[a])) for x in part["cuts"][a]) for a in range(2)]
    lines = {}
    for a in range(2):
        for k in cuts[a]:
            on = np.abs(nodes[:, a] - ax[a][k]) <= 1e-9
            ends = [u[0, k], u[-1, k]] if a == 0 else [u[k, 0], u[k, -1]]
            t = np.concatenate([[lo[1 - a]], nodes[on, 1 - a], [hi[1 - a]]])
            z = np.concatenate([[ends[0]], values[on], [ends[1]]])
            kern = lambda p, q: np.sqrt(1.0 + (part["rbf_eps"] * (p[:, None] - q[None, :])) ** 2)  # noqa: E731
            lines[a, k] = kern(ax[1 - a], t) @ np.linalg.solve(kern(t, t), z)
    for (a, k), v in lines.items():
        if a == 0:
            u[1:-1, k] = v[1:-1]
        else:
            u[k, 1:-1] = v[1:-1]
    for i in cuts[0]:
        for j in cuts[1]:
            u[j, i] = 0.5 * (lines[0, i][j] + lines[1, j][i])
    cx, cy = 0.5 / dx[0] ** 2, 0.5 / dx[1] ** 2
    W_, E_ = cx - b[..., 0] / (2 * dx[0]), cx + b[..., 0] / (2 * dx[0])
    S_, N_ = cy - b[..., 1] / (2 * dx[1]), cy + b[..., 1] / (2 * dx[1])
    C_ = -2 * cx - 2 * cy + c
    ix, iy = [0] + cuts[0] + [n[0] - 1], [0] + cuts[1] + [n[1] - 1]
    for i0, i1 in zip(ix, ix[1:]):
        for j0, j1 in zip(iy, iy[1:]):
            m, rows = i1 - i0 - 1, range(j0 + 1, j1)
            s = slice(i0 + 1, i1)
            G, y = np.zeros((m, m)), np.zeros(m)
            hold = []
            for j in rows:  # block elimination upwards, one grid row at a time
                A = np.diag(C_[j, s]) + np.diag(W_[j, s][1:], -1) + np.diag(E_[j, s][:-1], 1)
                r = f[j, s].copy()
                r[0] -= W_[j, i0 + 1] * u[j, i0]
                r[-1] -= E_[j, i1 - 1] * u[j, i1]
                if j == j0 + 1:
                    r -= S_[j, s] * u[j0, s]
                else:
                    A -= S_[j, s][:, None] * G
                    r -= S_[j, s] * y
                up = np.diag(N_[j, s]) if j < j1 - 1 else np.zeros((m, m))
                if j == j1 - 1:
                    r -= N_[j, s] * u[j1, s]
                sol = np.linalg.solve(A, np.concatenate([up, r[:, None]], axis=1))
                G, y = sol[:, :m], sol[:, m]
                hold.append((G, y))
            v = np.zeros(m)
            for j, (G, y) in zip(reversed(rows), reversed(hold)):
                v = y - G @ v
                u[j, s] = v
    return u


def _exact_grids(case, seed):
    pd, grid, u = _grids_input(case, seed)
    D, u = grid["dim"], u.double()
    dx = [(grid["hi"][d] - grid["lo"][d]) / (grid["n"][d] - 1) for d in range(D)]
    grad, lap = [], 0.0
    for d in range(D):
        a = u.movedim(D - 1 - d, 0)
        g, l2 = torch.empty_like(a), torch.empty_like(a)
        g[1:-1], l2[1:-1] = a[2:] - a[:-2], a[2:] - 2 * a[1:-1] + a[:-2]
        g[0], g[-1] = -3 * a[0] + 4 * a[1] - a[2], 3 * a[-1] - 4 * a[-2] + a[-3]
        l2[0], l2[-1] = 2 * a[0] - 5 * a[1] + 4 * a[2] - a[3], 2 * a[-1] - 5 * a[-2] + 4 * a[-3] - a[-4]
        grad.append((g / (2 * dx[d])).movedim(0, D - 1 - d).contiguous())
        lap = lap + (l2 / dx[d] ** 2).movedim(0, D - 1 - d)
    ax = [torch.as_tensor(grid["lo"][d] + np.arange(grid["n"][d]) * dx[d]).cuda() for d in range(D)]
    mesh = torch.meshgrid(*ax[::-1], indexing="ij")
    x = torch.stack([t.reshape(-1) for t in mesh[::-1]], dim=1)
    U, gU, lU = _u_and_derivatives(pd, x)
    b = x @ torch.tensor(pd["B"], dtype=torch.float64, device="cuda").T
    c = pd["c_a"] + pd["c_b"] * (x * x).sum(1)
    f = 0.5 * lU + (b * gU).sum(1) + c * U
    adv = sum(b[:, d] * grad[d].reshape(-1) for d in range(D))
    resid = f - (0.5 * lap.reshape(-1) + adv + c * u.reshape(-1))
    return {"grad": grad, "resid": resid.reshape(u.shape)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "stage2":
        return _exact_stage2(case, seed)
    if kind == "grids":
        return _exact_grids(case, seed)
    # the walks' steps one after the other: only where they are few and the paths fit memory
    if kind == "solve" and case["problem"] != "ball2" and case["exit"] == "bridge":
        side = {"unit": 1.0, "square4": 4.0}.get(case["problem"], 2.0) / (1.41 if case["problem"] == "paper" else 1.0)
        if side ** 2 / case["dt"] <= 4000 and case["nodes"] * case["paths"] <= 2_000_000:
            return _exact_solve(case, seed)
    return None
