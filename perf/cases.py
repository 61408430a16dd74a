"""The work this library is measured on: one case per use of its public entry points.

A case is a dict of plain values.  `op` names the path:

  spmv      y = A x through a plan kept for the matrix
  spmm      Y = A X likewise
  step      one differentiation step (forward, and both gradients) on a pattern whose context is kept
  pattern   the same step on a pattern the program has not used before: the context is part of the pass
  batch     many independent products in one Batched.run()
  assemble  triplets to canonical CSR
  reorder   degree order of a matrix and the symmetric permutation by it

`matrix` names the structure: "uniform" (a fixed number of random columns per row), "powerlaw"
(Zipf-Mandelbrot row lengths, columns drawn by weights of the same law), "ragged" (the same law
with empty rows), "stencil27" / "stencil5" (grids of odd and even sizes).
"""
import functools
import math

import numpy as np
import torch

import paper_1302_1078_amd as spx
from paper_1302_1078_amd.batch import Batched

DEV = "cuda"
TYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
SIZE = {"f64": 8, "f32": 4, "bf16": 2}
LMAX = 20_000  # longest row of the power laws


def listed():
    return [
        # the smallest call: 100,000 nonzeros in L2, launch and call latency
        {"name": "spmv-small", "op": "spmv", "matrix": "uniform", "m": 10_000, "n": 10_000, "mean": 10.0,
         "values": "f64", "plan": "default"},
        # an iterative solver or ranking iteration on a skewed graph, 16.8 M nonzeros
        {"name": "spmv-powerlaw", "op": "spmv", "matrix": "powerlaw", "m": 1 << 20, "n": 1 << 20, "mean": 16.0,
         "values": "f64", "plan": "hot"},
        # a grid solver that keeps its matrix in reduced precision, 55.7 M nonzeros
        {"name": "spmv-stencil", "op": "spmv", "matrix": "stencil27", "nx": 128, "ny": 128, "nz": 128,
         "values": "bf16", "plan": "default"},
        # several right-hand sides at once on the skewed graph
        {"name": "spmm-powerlaw", "op": "spmm", "matrix": "powerlaw", "m": 1 << 20, "n": 1 << 20, "mean": 16.0,
         "k": 16, "values": "f64", "plan": "default"},
        # block Krylov on the grid, rows ordered by band
        {"name": "spmm-stencil", "op": "spmm", "matrix": "stencil27", "nx": 128, "ny": 128, "nz": 128, "k": 32,
         "values": "f32", "plan": "banded"},
        # a rectangular matrix with empty rows, an odd number of right-hand sides, BF16 values
        {"name": "spmm-ragged", "op": "spmm", "matrix": "ragged", "m": 200_003, "n": 150_001, "mean": 12.0, "k": 5,
         "values": "bf16", "plan": "default"},
        # learning edge weights: one vector, 10.5 M nonzeros
        {"name": "step-vector", "op": "step", "matrix": "powerlaw", "m": 1 << 19, "n": 1 << 19, "mean": 20.0, "k": 1,
         "values": "f32", "mode": 0},
        # the same with several features per vertex
        {"name": "step-wide", "op": "step", "matrix": "powerlaw", "m": 1 << 18, "n": 1 << 18, "mean": 20.0, "k": 16,
         "values": "f32", "mode": 0},
        # a step on a subgraph sampled for it: index, map and plans are built for one use
        {"name": "pattern-step", "op": "pattern", "matrix": "powerlaw", "m": 131_072, "n": 131_072, "mean": 20.0,
         "k": 1, "values": "f32", "mode": 0},
        # many small and medium systems served together
        {"name": "batch", "op": "batch", "count": 48, "rmin": 1_000, "rmax": 200_000, "values": "f32"},
        # reading a graph: shuffled triplets with repeats
        {"name": "assemble", "op": "assemble", "matrix": "powerlaw", "m": 1 << 19, "n": 1 << 19, "mean": 16.0},
        # relabelling a graph so that its most-used vertices lie together
        {"name": "reorder", "op": "reorder", "matrix": "powerlaw", "m": 300_007, "n": 300_007, "mean": 16.0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["spmv", "spmv", "spmm", "spmm", "step", "step", "pattern", "batch", "assemble", "reorder"])
    if op == "batch":
        return {"op": op, "count": rng.randint(4, 48), "rmin": rng.choice([300, 1_000, 3_000]),
                "rmax": _log(rng, 20_000, 200_000), "values": rng.choice(["f64", "f32", "bf16"])}
    c = {"op": op}
    if op in ("spmv", "spmm") and rng.random() < 0.4:
        c["matrix"] = "stencil27"
        for d in ("nx", "ny", "nz"):
            c[d] = _log(rng, 10, 128)
    else:
        c["matrix"] = rng.choice(["uniform", "powerlaw", "ragged"])
        c["m"] = _log(rng, 3_000, {"spmv": 1 << 20, "spmm": 1 << 20, "step": 1 << 18, "pattern": 131_072,
                                   "assemble": 1 << 19, "reorder": 300_007}[op])
        c["n"] = c["m"] if op == "reorder" or rng.random() < 0.6 else max(3_000, int(c["m"] * rng.uniform(0.5, 1.0)))
        c["mean"] = round(rng.uniform(4.0, 16.0), 2)
    if op in ("spmv", "spmm"):
        c["values"] = rng.choice(["f64", "f32", "bf16"])
        plans = ["default", "default", "none"]
        if c["matrix"] == "stencil27":
            plans.append("banded")
        elif op == "spmv":
            plans.append("hot")
        c["plan"] = rng.choice(plans)
    if op == "spmm":
        c["k"] = rng.choice([2, 3, 4, 5, 8, 11, 16, 16]) if c.get("m", 0) > 200_000 else rng.choice(
            [2, 3, 4, 5, 7, 8, 13, 16, 24, 32])
    if op in ("step", "pattern"):
        c["k"] = rng.choice([1, 1, 2, 3, 4, 8, 12, 16])
        c["values"] = rng.choice(["f64", "f32"])
        c["mode"] = rng.choice([0, 0, 0, 1])
    return c


# ---------------------------------------------------------------- matrices

@functools.lru_cache(maxsize=None)
def _shift(alpha, lmax, mean):
    """q of the Zipf-Mandelbrot survival function ((1 + q) / (l + q))^(alpha - 1) with this mean."""
    l = np.arange(1, lmax + 1, dtype=np.float64)
    lo, hi = 0.0, 1e6
    for _ in range(80):
        q = 0.5 * (lo + hi)
        if np.sum(((1.0 + q) / (l + q)) ** (alpha - 1.0)) < mean:
            lo = q
        else:
            hi = q
    return 0.5 * (lo + hi)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _lengths(g, count, alpha, lmax, mean):
    """The law's quantiles in random order: the lengths vary in place only, so that a case has one nonzero count."""
    q = _shift(alpha, lmax, mean)
    u = (torch.randperm(count, generator=g, device=DEV).double() + 0.5) / count
    return ((1.0 + q) * u ** (-1.0 / (alpha - 1.0)) - q).floor().clamp_(1, lmax).to(torch.int64)


def _uniform(g, *shape, dtype=torch.float64):
    return (2.0 * torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64) - 1.0).to(dtype)


def _draw_entries(g, kind, m, n, mean, alpha=2.0):
    """Row and column of each entry, all distinct, rows and columns ascending."""
    if kind == "uniform":
        rows = torch.arange(m, device=DEV).repeat_interleave(int(round(mean)))
        cols = torch.randint(0, n, (rows.numel(),), generator=g, device=DEV)
    else:
        lmax = min(LMAX, n // 4)
        empty = int(kind == "ragged")  # one off each length of a longer mean: the shortest rows hold nothing
        lens = _lengths(g, m, alpha, lmax, mean + empty) - empty
        weight = _lengths(g, n, alpha, lmax, mean).double().cumsum(0)
        rows = torch.arange(m, device=DEV).repeat_interleave(lens)
        u = torch.rand(rows.numel(), generator=g, device=DEV, dtype=torch.float64) * weight[-1]
        cols = torch.searchsorted(weight, u, right=True).clamp_(max=n - 1)
    keys = rows * n + cols
    while True:  # a column drawn twice in a row gives way to a uniform one
        keys = torch.sort(keys)[0]
        twice = torch.nonzero(keys[1:] == keys[:-1]).flatten()
        if not twice.numel():
            return keys // n, keys % n
        keys[twice] = keys[twice] // n * n + torch.randint(0, n, (twice.numel(),), generator=g, device=DEV)


def _grid_entries(dims, reach):
    """Entries of a grid operator: every neighbour within `reach` steps (axes together), rows and columns ascending."""
    m = math.prod(dims)
    idx = torch.arange(m, device=DEV)
    at, rest = [], idx
    for d in reversed(dims):
        at.append(rest % d)
        rest = rest // d
    at.reverse()
    cols, ok = [], []
    offsets = [()]
    for _ in dims:
        offsets = [o + (s,) for o in offsets for s in (-1, 0, 1)]
    for o in offsets:
        if sum(map(abs, o)) > reach:
            continue
        good, shift = torch.ones(m, dtype=torch.bool, device=DEV), 0
        for a, s, d in zip(at, o, dims):
            good &= (a + s >= 0) & (a + s < d)
            shift = shift * d + s
        cols.append(idx + shift)
        ok.append(good)
    ok = torch.stack(ok, 1)
    return idx[:, None].expand_as(ok)[ok], torch.stack(cols, 1)[ok]


def _sorted_entries(g, c):
    if c["matrix"] == "stencil27":
        rows, cols = _grid_entries((c["nz"], c["ny"], c["nx"]), 3)
        return rows, cols, c["nx"] * c["ny"] * c["nz"], c["nx"] * c["ny"] * c["nz"]
    if c["matrix"] in ("stencil5", "stencil7"):
        rows, cols = _grid_entries(c["grid"], 1)
        return rows, cols, math.prod(c["grid"]), math.prod(c["grid"])
    m, n = c["m"], c["n"]
    return (*_draw_entries(g, c["matrix"], m, n, c["mean"], c.get("alpha", 2.0)), m, n)


def _rowptr(rows, m):
    rp = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(rows, minlength=m), 0, out=rp[1:])
    return rp.to(torch.int32)


def _matrix(g, c, values):
    """(CSR with values of the type, row of each nonzero)."""
    rows, cols, m, n = _sorted_entries(g, c)
    return spx.CSR(_rowptr(rows, m), cols.to(torch.int32), _uniform(g, rows.numel(), dtype=TYPES[values]),
                   (m, n)), rows


def _xtype(values):
    return torch.float64 if values == "f64" else torch.float32


def _dense(g, rows, k, dtype):
    return _uniform(g, rows, dtype=dtype) if k == 1 else _uniform(g, rows, k, dtype=dtype)


# ---------------------------------------------------------------- the cases' inputs

def _specs(c):
    """The matrices of a batch: a quarter 2D 5-point grids, a quarter 3D 7-point, half power laws; rows spread
    over their logarithm, the widths 1, 4 and 16 in turn."""
    out = []
    for i in range(c["count"]):
        f = ((i * 0.6180339887) + 0.31) % 1.0
        rows = int(round(c["rmin"] * (c["rmax"] / c["rmin"]) ** f))
        k = (1, 4, 16)[i % 3]
        if i % 4 == 0:
            s = max(2, round(math.sqrt(rows)))
            out.append({"matrix": "stencil5", "grid": (s, s), "k": k})
        elif i % 4 == 2:
            s = max(2, round(rows ** (1 / 3)))
            out.append({"matrix": "stencil7", "grid": (s, s, s), "k": k})
        else:
            out.append({"matrix": "powerlaw", "m": rows, "n": rows, "mean": 8.0 + 2 * (i % 13), "alpha": 2.2, "k": k})
    return out


def _inputs(c, seed):
    """What a pass reads, as plain tensors and CSR arrays: no plan, no call into the library."""
    g = _gen(seed)
    op = c["op"]
    if op == "batch":
        mats, rows, Xs = [], [], []
        for s in _specs(c):
            A, r = _matrix(g, s, c["values"])
            mats.append(A)
            rows.append(r)
            Xs.append(_dense(g, A.n, s["k"], _xtype(c["values"])))
        return {"mats": mats, "rows": rows, "Xs": Xs}
    if op == "assemble":
        rows, cols = _draw_entries(g, c["matrix"], c["m"], c["n"], c["mean"])
        # one entry in 32 is given twice
        again = torch.randint(0, rows.numel(), (rows.numel() // 32,), generator=g, device=DEV)
        order = torch.randperm(rows.numel() + again.numel(), generator=g, device=DEV)
        rows, cols = (torch.cat([t, t[again]])[order] for t in (rows, cols))
        return {"r": rows.to(torch.int32), "c": cols.to(torch.int32), "v": _uniform(g, rows.numel())}
    if op == "reorder":
        A, rows = _matrix(g, c, "f64")
        return {"A": A, "rows": rows}
    A, rows = _matrix(g, c, c["values"])
    k, xt = c.get("k", 1), _xtype(c["values"])
    d = {"A": A, "rows": rows, "x": _dense(g, A.n, k, xt)}
    if op in ("step", "pattern"):
        d["dy"] = _dense(g, A.m, k, xt)
    return d


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["op"] = c["op"]
    s.pop("rows", None)
    if c["op"] in ("spmv", "spmm"):
        A, k = s["A"], c.get("k", 1)
        if c["plan"] == "none":
            s["plan"] = None
        elif c["plan"] == "banded":
            s["plan"] = spx.Plan.for_matrix(A, spx.banded_opts(A, k, A.values.dtype))
        else:
            s["plan"] = spx.Plan.for_matrix(A, k=k)
            if c["plan"] == "hot":
                s["plan"].attach_hot_x(A, 65_536, s["x"].dtype)
    elif c["op"] in ("step", "pattern"):
        s["k"], s["mode"] = c["k"], c["mode"]
        if c["op"] == "step":
            s["grad"] = spx.GradContext(s["A"], mode=c["mode"], k=c["k"])
        s["w"] = s["A"].values.clone().requires_grad_()
        s["x"].requires_grad_()
    elif c["op"] == "batch":
        s["batch"] = Batched(s["mats"], s["Xs"])
    elif c["op"] == "assemble":
        s["m"], s["n"] = c["m"], c["n"]
    return s


def run(state):
    s = state
    op = s["op"]
    if op == "spmv":
        return spx.spmv(s["A"], s["x"], plan=s["plan"])
    if op == "spmm":
        return spx.spmm(s["A"], s["x"], plan=s["plan"])
    if op in ("step", "pattern"):
        g = s["grad"] if op == "step" else spx.GradContext(s["A"], mode=s["mode"], k=s["k"])
        y = spx.spmv_autograd(s["w"], s["x"], g)
        dw, dx = torch.autograd.grad(y, (s["w"], s["x"]), s["dy"])
        return y, dw, dx
    if op == "batch":
        return s["batch"].run()
    if op == "assemble":
        A = spx.from_coo(s["m"], s["n"], s["r"], s["c"], s["v"])
        return A.rowptr, A.colind, A.values
    perm = spx.degree_order(s["A"])
    B = spx.permute(s["A"], perm)
    return perm, B.rowptr, B.colind, B.values


# ---------------------------------------------------------------- work and 64-bit results

def _shape(c):
    """(rows, columns, nonzeros) of a case's matrix, the nonzeros as the law gives them."""
    if c["matrix"] == "stencil27":
        d = (c["nx"], c["ny"], c["nz"])
        return math.prod(d), math.prod(d), math.prod(3 * x - 2 for x in d)
    if c["matrix"] in ("stencil5", "stencil7"):
        d, m = c["grid"], math.prod(c["grid"])
        return m, m, m + 2 * sum(m // x * (x - 1) for x in d)
    return c["m"], c["n"], int(c["m"] * (round(c["mean"]) if c["matrix"] == "uniform" else c["mean"]))


def _product_work(c, values):
    m, n, nnz = _shape(c)
    k, sv, sx = c.get("k", 1), SIZE[values], 8 if values == "f64" else 4
    return (sv + 4) * nnz + sx * k * (m + n) + 4 * (m + 1), 2.0 * nnz * k


def work(case):
    c = case
    op = c["op"]
    if op == "batch":
        per = [_product_work(s, c["values"]) for s in _specs(c)]
        return {"bytes": sum(p[0] for p in per), "flops": sum(p[1] for p in per)}
    m, n, nnz = _shape(c)
    if op == "assemble":
        given = nnz + nnz // 32
        return {"bytes": 16 * given + 12 * nnz + 4 * (m + 1), "flops": 0}
    if op == "reorder":
        return {"bytes": 2 * (12 * nnz + 4 * (m + 1)) + 4 * m, "flops": 0}
    b, f = _product_work(c, c["values"])
    if op in ("step", "pattern"):
        # the pattern and values are read, y, dw and dx written; x and dy are read
        sx = SIZE[c["values"]]
        return {"bytes": b + sx * nnz + sx * c["k"] * (m + n), "flops": 3.0 * f}
    return {"bytes": b, "flops": f}


def _gathered(out_rows, to, frm, v, X):
    """out[to] += v * X[frm] in 64 bits, a few columns at a time."""
    out = torch.zeros((out_rows,) + tuple(X.shape[1:]), dtype=torch.float64, device=DEV)
    if X.dim() == 1:
        return out.index_add_(0, to, v * X[frm])
    for t in range(0, X.shape[1], 4):
        out[:, t:t + 4] = torch.zeros((out_rows, X[:, t:t + 4].shape[1]), dtype=torch.float64, device=DEV).index_add_(
            0, to, v[:, None] * X[frm, t:t + 4])
    return out


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    op = c["op"]
    if op == "batch":
        return [_gathered(A.m, r, A.colind.long(), A.values.double(), X.double())
                for A, r, X in zip(s["mats"], s["rows"], s["Xs"])]
    if op == "assemble":
        n = c["n"]
        keys, at = torch.unique(s["r"].long() * n + s["c"].long(), return_inverse=True)
        values = torch.zeros(keys.numel(), dtype=torch.float64, device=DEV).index_add_(0, at, s["v"])
        return _rowptr(keys // n, c["m"]), (keys % n).to(torch.int32), values
    A, rows = s["A"], s["rows"]
    cols = A.colind.long()
    if op == "reorder":
        perm = torch.sort(torch.bincount(cols, minlength=A.n), descending=True, stable=True)[1]
        label = torch.empty_like(perm)
        label[perm] = torch.arange(A.n, device=DEV)
        keys, order = torch.sort(label[rows] * A.n + label[cols])
        return (perm.to(torch.int32), _rowptr(keys // A.n, A.m), (keys % A.n).to(torch.int32), A.values[order])
    v, x = A.values.double(), s["x"].double()
    y = _gathered(A.m, rows, cols, v, x)
    if op in ("spmv", "spmm"):
        return y
    dy = s["dy"].double()
    if dy.dim() == 1:
        dw = dy[rows] * x[cols]
    else:
        dw = torch.zeros_like(v)
        for t in range(dy.shape[1]):
            dw += dy[rows, t] * x[cols, t]
    return y, dw, _gathered(A.n, cols, rows, v, dy)
