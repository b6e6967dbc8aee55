"""The work that programs built on this library have it do, as cases to be timed.

Every case goes through the public Python calls. Matrices and vectors are made
on the GPU from the seed alone, with the distributions of the package's own
synthetic inputs: R-MAT graphs (relabelled, U[0, 1] weights), uniform rows,
Pareto rows, the 7-point stencil, pruned fully-connected layers.

A case's "call" names the entry point:
  run       y = Matrix.run(x): one adaptive product, x dense or a list
  batch     Matrix.run_batch: many sparse vectors at once
  forward   Matrix.spmv_batch: a pruned layer at inference
  train     sparse_linear forward and both gradients
  bfs       Matrix.bfs: levels of a whole search
  pagerank  Matrix.pagerank: incremental PageRank to convergence
"""
from __future__ import annotations

import math

import torch

import paper_2006_16767_amd as spx
from paper_2006_16767_amd.autograd import sparse_linear

DEV = "cuda"
TORCH = {"f32": torch.float32, "f64": torch.float64, "i32": torch.int32, "minplus": torch.float32}
SIZE = {"f32": 4, "f64": 8, "i32": 4, "minplus": 4, "bool": 1}


def listed():
    graph = {"matrix": "rmat", "scale": 20, "degree": 16}
    return [
        # one small system, solved again and again: launch latency counts
        {"name": "small_dense", "call": "run", "matrix": "uniform", "m": 4096, "n": 4096, "per_row": 16, "dtype": "f32",
         "x": "dense"},
        # graph products as the frontier grows: a seed set ...
        {"name": "graph_x10", "call": "run", **graph, "dtype": "f32", "x": "sparse", "nnz_x": 10},
        # ... an early round ...
        {"name": "graph_x3834", "call": "run", **graph, "dtype": "f32", "x": "sparse", "nnz_x": 3834},
        # ... a wide one ...
        {"name": "graph_x73282", "call": "run", **graph, "dtype": "f32", "x": "sparse", "nnz_x": 73282},
        # ... and half of the graph
        {"name": "graph_x524288", "call": "run", **graph, "dtype": "f32", "x": "sparse", "nnz_x": 524288},
        # the matrix product of a stencil solver's iteration, single precision
        {"name": "stencil_f32", "call": "run", "matrix": "stencil", "k": 128, "dtype": "f32", "x": "dense"},
        # the same in double precision, on a grid whose side is odd
        {"name": "stencil_f64_odd", "call": "run", "matrix": "stencil", "k": 101, "dtype": "f64", "x": "dense"},
        # many queries against one graph, densities over four decades
        {"name": "batch_graph", "call": "batch", "matrix": "rmat", "scale": 18, "degree": 32, "B": 512, "dtype": "f32"},
        # a pruned layer at inference
        {"name": "layer_forward", "call": "forward", "m": 16384, "n": 4096, "p": 0.05, "B": 64, "dtype": "f32"},
        # one training step of that layer: output, input and weight gradients
        {"name": "layer_train", "call": "train", "m": 16384, "n": 4096, "p": 0.05, "B": 64, "dtype": "f32"},
        # a whole search of a graph
        {"name": "bfs", "call": "bfs", **graph, "dtype": "bool"},
        # a whole ranking of a graph, to convergence
        {"name": "pagerank", "call": "pagerank", **graph, "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, lo, hi):
    scale = rng.randint(lo, hi)
    return {"matrix": "rmat", "scale": scale, "degree": rng.randint(4, 16 if scale >= 19 else 32)}


def draw(rng):
    call = rng.choice(["run", "run", "run", "run", "batch", "forward", "train", "bfs", "pagerank"])
    if call == "run":
        kind = rng.choice(["rmat", "rmat", "uniform", "powerlaw", "stencil"])
        dtype = rng.choice(["f32", "f32", "f32", "f64", "i32", "minplus", "bool"])
        if kind == "rmat":
            c = _draw_graph(rng, 12, 20)
            n = 1 << c["scale"]
        elif kind == "uniform":
            n = _log(rng, 1000, 200000)
            c = {"matrix": "uniform", "m": _log(rng, 1000, 200000), "n": n, "per_row": rng.randint(3, 64)}
        elif kind == "powerlaw":
            n = _log(rng, 1000, 50000)
            c = {"matrix": "powerlaw", "m": _log(rng, 2000, 100000), "n": n, "mean": rng.randint(5, 40)}
        else:
            dtype = rng.choice(["f32", "f64"])
            c = {"matrix": "stencil", "k": rng.randint(20, 120)}
            n = c["k"] ** 3
        c = {"call": "run", **c, "dtype": dtype}
        if dtype != "bool" and rng.random() < (0.7 if kind == "stencil" else 0.25):
            return {**c, "x": "dense"}
        return {**c, "x": "sparse", "nnz_x": max(1, min(n // 2, _log(rng, 1e-5 * n + 1, 0.5 * n)))}
    if call == "batch":
        if rng.random() < 0.5:
            c = _draw_graph(rng, 12, 17)
        else:
            c = {"matrix": "powerlaw", "m": _log(rng, 5000, 100000), "n": _log(rng, 5000, 50000), "mean": rng.randint(10, 40)}
        return {"call": "batch", **c, "B": _log(rng, 8, 400), "dtype": "f32"}
    if call in ("forward", "train"):
        return {"call": call, "m": _log(rng, 256, 16384), "n": _log(rng, 256, 4096), "p": rng.choice([0.02, 0.05, 0.1]) / 2,
                "B": _log(rng, 1, 64), "dtype": rng.choice(["f32", "f32", "f32", "f64"])}
    c = _draw_graph(rng, 12, 19)
    return {"call": call, **c, "dtype": "bool" if call == "bfs" else rng.choice(["f32", "f64"])}


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 16767)
    return g


def _csr(m, n, rows, cols):
    """Row pointers and column indices of distinct (row, column) pairs."""
    key = torch.unique(rows * n + cols)
    rows = torch.div(key, n, rounding_mode="floor")
    ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=m), 0)
    return ptr.to(torch.int32), (key - rows * n).to(torch.int32)


def _rmat(c, g):
    """Quadrants (0.57, 0.19, 0.19, 0.05), duplicates removed, vertices
    relabelled; entry (i, j) is the edge j -> i."""
    nv, e = 1 << c["scale"], c["degree"] << c["scale"]
    src = torch.zeros(e, dtype=torch.int64, device=DEV)
    dst = torch.zeros(e, dtype=torch.int64, device=DEV)
    for _ in range(c["scale"]):
        r = torch.rand(e, generator=g, device=DEV)
        src = src * 2 + (r >= 0.76)
        dst = dst * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    perm = torch.randperm(nv, generator=g, device=DEV)
    return (nv, nv) + _csr(nv, nv, perm[dst], perm[src])


def _uniform(c, g):
    m, n = c["m"], c["n"]
    rows = torch.arange(m, device=DEV).repeat_interleave(min(c["per_row"], n))
    cols = torch.randint(0, n, (rows.numel(),), generator=g, device=DEV)
    return (m, n) + _csr(m, n, rows, cols)


def _powerlaw(c, g):
    """Pareto(1.5) row lengths, uniform columns."""
    m, n = c["m"], c["n"]
    u = torch.rand(m, generator=g, device=DEV, dtype=torch.float64).clamp_min(1e-9)
    lens = torch.clamp(torch.ceil(c["mean"] / 3.0 * u ** (-1 / 1.5)), max=n // 4).to(torch.int64)
    rows = torch.repeat_interleave(torch.arange(m, device=DEV), lens)
    cols = torch.randint(0, n, (rows.numel(),), generator=g, device=DEV)
    return (m, n) + _csr(m, n, rows, cols)


def _stencil(c, g):
    k = c["k"]
    i = torch.arange(k ** 3, device=DEV)
    x, y, z = i % k, torch.div(i, k, rounding_mode="floor") % k, torch.div(i, k * k, rounding_mode="floor")
    cols = torch.stack([i - k * k, i - k, i - 1, i, i + 1, i + k, i + k * k], 1)
    on = torch.stack([z > 0, y > 0, x > 0, i >= 0, x < k - 1, y < k - 1, z < k - 1], 1)
    ptr = torch.zeros(k ** 3 + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(on.sum(1), 0)
    return k ** 3, k ** 3, ptr.to(torch.int32), cols[on].to(torch.int32)


def _layer(c, g):
    """A fixed share of the weights is kept (the gradient's length is the
    program's own), each weight with the same chance."""
    m, n = c["m"], c["n"]
    kept = torch.randperm(m * n, generator=g, device=DEV)[: round(c["p"] * m * n)]
    rows = torch.div(kept, n, rounding_mode="floor")
    return (m, n) + _csr(m, n, rows, kept - rows * n)


def _values(kind, dtype, shape, g):
    if dtype == "bool":
        return None
    if dtype == "i32":
        return torch.randint(-4, 5, (shape,), generator=g, device=DEV, dtype=torch.int32)
    v = torch.rand(shape, generator=g, device=DEV, dtype=TORCH[dtype])
    return v if kind in ("rmat", "powerlaw") else 2 * v - 1


def _matrix(c, g):
    """(m, n, row_ptr, col_idx, vals, entry rows)."""
    kind = c.get("matrix", "layer")
    m, n, ptr, col = {"rmat": _rmat, "uniform": _uniform, "powerlaw": _powerlaw, "stencil": _stencil, "layer": _layer}[kind](c, g)
    if kind == "stencil":
        row = torch.repeat_interleave(torch.arange(m, device=DEV), torch.diff(ptr))
        vals = torch.where(row == col, 6.0, -1.0).to(TORCH[c["dtype"]])
    elif kind == "layer":
        vals = 0.02 * torch.randn(col.numel(), generator=g, device=DEV, dtype=TORCH[c["dtype"]])
    else:
        vals = _values(kind, c["dtype"], col.numel(), g)
    return m, n, ptr, col, vals


def _inputs(c, seed):
    g = _gen(seed)
    m, n, ptr, col, vals = _matrix(c, g)
    d = {"m": m, "n": n, "ptr": ptr, "col": col, "vals": vals}
    call, dt = c["call"], c["dtype"]
    if call == "run":
        if c["x"] == "dense":
            d["x"] = _values("dense", dt, n, g)
        else:
            idx = torch.sort(torch.randperm(n, generator=g, device=DEV)[: c["nnz_x"]])[0].to(torch.int32)
            d["x"] = (idx, _values(c["matrix"], dt, c["nnz_x"], g))
    elif call == "batch" and c["matrix"] == "rmat":
        # densities log-uniform in [1e-4, 0.5], uniform supports
        dens = 10.0 ** (-4.0 + (math.log10(0.5) + 4.0) * torch.rand(c["B"], generator=g, device=DEV))
        idx = [torch.nonzero(torch.rand(n, generator=g, device=DEV) < p)[:, 0] for p in dens.tolist()]
        d["vec_ptr"] = torch.tensor([0] + [i.numel() for i in idx], device=DEV).cumsum(0).to(torch.int32)
        d["idx"] = torch.cat(idx).to(torch.int32)
        d["val"] = _values("rmat", dt, d["idx"].numel(), g)
    elif call == "batch":
        # rows of the data matrix itself
        rows = torch.sort(torch.randperm(m, generator=g, device=DEV)[: c["B"]])[0]
        lens = (ptr[1:] - ptr[:-1])[rows].to(torch.int64)
        d["vec_ptr"] = torch.cat([lens.new_zeros(1), lens.cumsum(0)]).to(torch.int32)
        at = torch.arange(int(lens.sum()), device=DEV) - torch.repeat_interleave(d["vec_ptr"][:-1].to(torch.int64) - ptr[rows], lens)
        d["idx"], d["val"] = col[at].contiguous(), vals[at].contiguous()
    elif call in ("forward", "train"):
        # activations after a rectifier: half to 95 % zeros, |N(0, 1)| elsewhere
        B = c["B"]
        zero = 0.5 + 0.45 * torch.arange(B, device=DEV)[:, None] / max(B - 1, 1)
        X = torch.randn((B, n), generator=g, device=DEV, dtype=TORCH[dt]).abs()
        d["X"] = torch.where(torch.rand((B, n), generator=g, device=DEV) < zero, torch.zeros_like(X), X)
        d["G"] = torch.randn((B, m), generator=g, device=DEV, dtype=TORCH[dt])
    elif call == "bfs":
        d["source"] = int(col.min())  # the lowest vertex with an out-edge
    return d


DTYPE = {"f32": spx.F32, "f64": spx.F64, "i32": spx.I32, "bool": spx.BOOL, "minplus": spx._lib.F32_MINPLUS}


def prepare(case, seed):
    d = _inputs(case, seed)
    d["call"] = case["call"]
    if case["call"] == "train":
        d["vals"].requires_grad_(True)
        d["X"].requires_grad_(True)
    d["M"] = spx.Matrix(d["ptr"], d["col"], d["vals"], d["m"], d["n"], DTYPE[case["dtype"]])
    return d


def run(s):
    M, call = s["M"], s["call"]
    if call == "run":
        return M.run(s["x"])
    if call == "batch":
        return M.run_batch(s["vec_ptr"], s["idx"], s["val"])
    if call == "forward":
        return M.spmv_batch(s["X"])
    if call == "train":
        Y = sparse_linear(M, s["X"], s["vals"])
        dX, dvals = torch.autograd.grad(Y, (s["X"], s["vals"]), s["G"])
        return Y.detach(), dX, dvals
    if call == "bfs":
        return M.bfs(s["source"])[0]
    return M.pagerank()[0]


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------
def _entries(c):
    kind = c.get("matrix", "layer")
    if kind == "rmat":  # about 4 % of the sampled edges are duplicates
        return 1 << c["scale"], 1 << c["scale"], 0.96 * (c["degree"] << c["scale"])
    if kind == "uniform":
        return c["m"], c["n"], float(c["m"]) * c["per_row"]
    if kind == "powerlaw":
        return c["m"], c["n"], float(c["m"]) * c["mean"]
    if kind == "stencil":
        return c["k"] ** 3, c["k"] ** 3, 7.0 * c["k"] ** 3 - 6.0 * c["k"] ** 2
    return c["m"], c["n"], c["p"] * c["m"] * c["n"]


def work(case):
    m, n, nnz = _entries(case)
    call = case["call"]
    vs = SIZE[case["dtype"]]
    a = nnz * (4 + (0 if case["dtype"] == "bool" else vs)) + 4 * (m + 1)
    if call == "run":
        if case["matrix"] == "stencil":  # the diagonals' values; their places are seven numbers
            dense = nnz * vs + (n + m) * vs
        else:
            dense = a + (n + m) * vs
        if case["x"] == "dense":
            return {"bytes": dense, "flops": 2 * nnz}
        eff = nnz * case["nnz_x"] / n  # entries in the columns that x lists
        ev = 0 if case["dtype"] == "bool" else vs
        lists = case["nnz_x"] * (12 + ev) + eff * (4 + ev) + m * vs
        return {"bytes": min(dense, lists), "flops": 2 * eff}
    if call == "batch":
        if case["matrix"] == "rmat":  # the mean of a log-uniform density
            share = (0.5 - 1e-4) / math.log(0.5 / 1e-4)
        else:
            share = case["mean"] / n
        B = case["B"]
        return {"bytes": a + B * n * share * (4 + vs) + B * m * vs, "flops": 2 * B * nnz * share}
    if call == "forward":
        return {"bytes": a + case["B"] * (m + n) * vs, "flops": 2 * nnz * case["B"]}
    if call == "train":
        # forward; backward reads the pattern again, both operands, and writes both gradients
        return {"bytes": 2 * a + case["B"] * (2 * m + 3 * n) * vs + nnz * vs, "flops": 6 * nnz * case["B"]}
    if call == "bfs":
        # per vertex a level, a pointer and at least the entry that reached it
        return {"bytes": 12 * n, "flops": nnz}
    # about 50 of the rounds see most of the graph active
    return {"bytes": 50 * (a + 6 * n * vs), "flops": 100 * nnz}


# ----------------------------------------------------------------------------
# the same results in 64 bits
# ----------------------------------------------------------------------------
def _product(d, x, row):
    return torch.zeros(d["m"], dtype=torch.float64, device=DEV).index_add_(0, row, d["vals"].double() * x[d["col"]])


def _exact_pagerank(d, row):
    n, damping = d["n"], 0.85
    eps = 1e-3 * (1.0 - damping) / max(1, n)
    W = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, d["col"], d["vals"].double())
    p = torch.zeros(n, dtype=torch.float64, device=DEV)
    r = torch.full((n,), (1.0 - damping) / n, dtype=torch.float64, device=DEV)
    for _ in range(10000):
        hot = r.abs() > eps
        p = p + torch.where(hot, r, 0.0)
        x = torch.where(hot & (W > 0), r / torch.where(W > 0, W, 1.0), 0.0)
        r = torch.where(hot, 0.0, r)
        if not bool((x != 0).any()):
            break
        r = r + damping * _product(d, x, row)
    return p


def exact(case, seed):
    call, dt = case["call"], case["dtype"]
    if call == "bfs" or dt in ("i32", "bool"):
        return None
    d = _inputs(case, seed)
    m, n = d["m"], d["n"]
    row = torch.repeat_interleave(torch.arange(m, device=DEV), torch.diff(d["ptr"]))
    d["col"] = d["col"].to(torch.int64)
    if call == "run":
        zero = math.inf if dt == "minplus" else 0.0
        if case["x"] == "dense":
            x = d["x"].double()
        else:
            x = torch.full((n,), zero, dtype=torch.float64, device=DEV)
            x[d["x"][0].to(torch.int64)] = d["x"][1].double()
        if dt == "minplus":
            y = torch.full((m,), zero, dtype=torch.float64, device=DEV)
            return y.scatter_reduce_(0, row, d["vals"].double() + x[d["col"]], "amin")
        return _product(d, x, row)
    if call == "batch":
        Y = torch.empty((case["B"], m), dtype=torch.float64, device=DEV)
        ptr = d["vec_ptr"].tolist()
        for b in range(case["B"]):
            x = torch.zeros(n, dtype=torch.float64, device=DEV)
            x[d["idx"][ptr[b]:ptr[b + 1]].to(torch.int64)] = d["val"][ptr[b]:ptr[b + 1]].double()
            Y[b] = _product(d, x, row)
        return Y
    if call in ("forward", "train"):
        A = torch.zeros((m, n), dtype=torch.float64, device=DEV)
        A[row, d["col"]] = d["vals"].double()
        X, G = d["X"].double(), d["G"].double()
        Y = X @ A.t().contiguous()
        if call == "forward":
            return Y
        return Y, G @ A, (G.t().contiguous() @ X)[row, d["col"]]
    return _exact_pagerank(d, row)
