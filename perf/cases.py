"""The calls whose speed this library is judged by, over the sizes it is used at.

``listed()`` names the fixed cases, ``draw(rng)`` gives one more of the same
ranges.  ``prepare`` makes on the GPU what a program holds before the call
(points, targets, output buffers, workspaces), ``run`` is one call through the
public entry points of ``paper_1308_1419_amd.tdmap``, ``work`` the bytes and
operations the call cannot do without, ``exact`` the same outputs in 64 bits
from plain torch.

Sizes are those of ``synth.WORKLOADS`` and of the tests, or generic ones
between them; ragged sizes are there because packed rows, tile edges and set
boundaries fall differently on them.
"""
import math

import numpy as np
import torch

from paper_1308_1419_amd import tdmap

DEV = "cuda"


def listed():
    return [
        # one small distance matrix per call (a few neighbours, one frame of
        # a trajectory): launch and host latency
        {"name": "edm_n1024_d3_full", "kind": "edm", "N": 1024, "d": 3, "layout": "full"},
        # an ordinary pair list in the condensed layout, ragged N, 2D points
        {"name": "edm_n4999_d2_packed", "kind": "edm", "N": 4999, "d": 2, "layout": "packed"},
        # the benchmark's step: the whole matrix of a large cloud
        {"name": "edm_n30000_d3_full", "kind": "edm", "N": 30000, "d": 3, "layout": "full"},
        # an interaction table without the diagonal, ragged N
        {"name": "edm_n20011_d4_strict", "kind": "edm", "N": 20011, "d": 4, "layout": "strict"},
        # a training step that differentiates through the distances: forward
        # and backward by autograd, at the size of one sample
        {"name": "autograd_n3001_d3", "kind": "autograd", "N": 3001, "d": 3},
        # the gradient alone, at the stress workload's size
        {"name": "backward_n20000_d3_packed", "kind": "backward", "N": 20000, "d": 3,
         "layout": "packed", "deterministic": True},
        # one iteration of metric multidimensional scaling: loss and gradient
        {"name": "stress_n20000_d3_packed", "kind": "stress", "N": 20000, "d": 3,
         "layout": "packed", "deterministic": True},
        # feature vectors of ordinary width, all pairs, BF16 products
        {"name": "gram_bf16_n100000_d64", "kind": "gram", "N": 100000, "d": 64,
         "precision": "bf16_gram"},
        # wider features at a ragged size, near-FP32 products
        {"name": "gram_bf16x3_n30011_d200", "kind": "gram", "N": 30011, "d": 200,
         "precision": "bf16x3_gram"},
        # many clouds of mixed sizes in one launch (the batched workload's
        # size range, a quarter of its sets)
        {"name": "batched_s1024_n64_4096_d3", "kind": "batched", "sets": 1024, "n_min": 64,
         "n_max": 4096, "d": 3},
        # thousands of molecule-sized sets, empty ones among them
        {"name": "batched_s3000_n0_139_d3", "kind": "batched", "sets": 3000, "n_min": 0,
         "n_max": 139, "d": 3},
        # exact FP32 distances of points with more features than the tiles
        # take (the paper's one-cell-per-thread launch)
        {"name": "cell_n8000_d16_full", "kind": "cell", "N": 8000, "d": 16, "rho": 16,
         "layout": "full"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["edm", "edm", "autograd", "backward", "stress", "gram", "batched", "cell"])
    layout = rng.choice(["full", "packed", "strict"])
    d = rng.randint(1, 4)
    if kind == "edm":
        return {"kind": kind, "N": _log(rng, 256, 30000), "d": d, "layout": layout}
    if kind == "autograd":
        return {"kind": kind, "N": _log(rng, 256, 8000), "d": d}
    if kind in ("backward", "stress"):
        return {"kind": kind, "N": _log(rng, 1000, 20000), "d": d, "layout": layout,
                "deterministic": rng.random() < 0.7}
    if kind == "gram":
        prec = rng.choice(["bf16_gram", "bf16x3_gram"])
        d = _log(rng, 8, 256)
        top = 100000 * min(1.0, math.sqrt(64 / d)) * (0.6 if prec == "bf16x3_gram" else 1.0)
        return {"kind": kind, "N": _log(rng, 500, top), "d": d, "precision": prec}
    if kind == "batched":
        n_max = _log(rng, 32, 4096)
        sets = _log(rng, 16, min(4096, 16 + 2.5e9 * 6 / n_max ** 2))
        return {"kind": kind, "sets": sets, "n_min": rng.choice([0, n_max // 4, n_max // 2]),
                "n_max": n_max, "d": d}
    return {"kind": "cell", "N": _log(rng, 500, 8000), "d": _log(rng, 5, 32),
            "rho": rng.choice([8, 16, 32]), "layout": rng.choice(["full", "packed"])}


# ---------------------------------------------------------------------------
# sizes
# ---------------------------------------------------------------------------

def _cells(N, layout):
    return N * (N - 1) // 2 if layout == "strict" else N * (N + 1) // 2


def _buffer(N, layout):
    """A buffer of the layout; the full one is zeroed, as its upper triangle
    is never written."""
    if layout == "full":
        return torch.zeros((N, N), dtype=torch.float32, device=DEV)
    return torch.empty(_cells(N, layout), dtype=torch.float32, device=DEV)


def _set_sizes(case):
    """Set sizes belong to the case, so that every seed has the same shapes."""
    rng = np.random.Generator(np.random.PCG64(1000 * case["sets"] + case["n_max"]))
    n = rng.integers(case["n_min"], case["n_max"], size=case["sets"], endpoint=True).astype(np.int64)
    point_off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    out_off = np.concatenate([[0], np.cumsum(n * (n + 1) // 2)]).astype(np.int64)
    return n, point_off, out_off


def _rows_per_block(N):
    return max(1, min(N, 40_000_000 // max(1, N)))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1308141900 + seed)
    return g


def _uniform(N, d, g):
    return torch.rand((N, d), dtype=torch.float32, device=DEV, generator=g)


def _features(N, d, g):
    """N(0, 1) features; one point in a hundred nearly repeats another."""
    X = torch.randn((N, d), dtype=torch.float32, device=DEV, generator=g)
    m = N // 100
    if m:
        perm = torch.randperm(N, device=DEV, generator=g)
        src = perm[m:2 * m]
        X[perm[:m]] = X[src] + 1e-4 * torch.randn((m, d), dtype=torch.float32, device=DEV,
                                                  generator=g)
    return X


def _pack(rows, N, layout, dtype):
    """The layout's buffer from `rows(r0, r1)`, which gives rows r0 .. r1 - 1
    over the columns 0 .. r1 - 1."""
    if layout == "full":
        out = torch.zeros((N, N), dtype=dtype, device=DEV)
    else:
        out = torch.empty(_cells(N, layout), dtype=dtype, device=DEV)
    step = _rows_per_block(N)
    for r0 in range(0, N, step):
        r1 = min(N, r0 + step)
        v = rows(r0, r1)
        if layout == "full":
            out[r0:r1, :r1] = torch.tril(v, diagonal=r0)
        else:
            strict = 1 if layout == "strict" else 0
            keep = torch.ones_like(v, dtype=torch.bool).tril_(diagonal=r0 - strict)
            a = _cells(r0, layout) if r0 else 0
            b = _cells(r1, layout)
            out[a:b] = v[keep]
    return out


def _targets(N, d, layout, X, g):
    """Distances of a disturbed copy of the points: what a fit is given."""
    Xp = X + 0.05 * torch.randn((N, d), dtype=torch.float32, device=DEV, generator=g)
    return _pack(lambda a, b: _dist(Xp, a, b), N, layout, torch.float32)


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    d = case["d"]
    if kind == "batched":
        _, po, oo = _set_sizes(case)
        S = case["sets"]
        return {"case": case, "X": _uniform(int(po[-1]), d, g),
                "po": torch.from_numpy(po).to(DEV), "oo": torch.from_numpy(oo).to(DEV),
                "out": torch.empty(int(oo[-1]), dtype=torch.float32, device=DEV),
                "ws": torch.empty(tdmap.tdmap_workspace_size(tdmap.OP_BATCHED, 0, d, S, 0, 0),
                                  dtype=torch.uint8, device=DEV)}
    N = case["N"]
    if kind == "gram":
        prec = tdmap.PRECISIONS[case["precision"]]
        return {"case": case, "X": _features(N, d, g), "out": _buffer(N, "packed"),
                "ws": torch.empty(tdmap.tdmap_workspace_size(tdmap.OP_EDM, N, d, 0, 0, prec),
                                  dtype=torch.uint8, device=DEV)}
    X = _uniform(N, d, g)
    if kind in ("edm", "cell"):
        return {"case": case, "X": X, "out": _buffer(N, case["layout"])}
    if kind == "autograd":
        dD = torch.randn(_cells(N, "packed"), dtype=torch.float32, device=DEV, generator=g)
        return {"case": case, "X": X.requires_grad_(True), "dD": dD}
    layout = case["layout"]
    st = {"case": case, "X": X, "dX": torch.empty((N, d), dtype=torch.float32, device=DEV)}
    if kind == "backward":
        op = tdmap.OP_BACKWARD
        shape = (N, N) if layout == "full" else (_cells(N, layout),)
        st["dD"] = torch.randn(shape, dtype=torch.float32, device=DEV, generator=g)
    else:
        op = tdmap.OP_STRESS
        st["delta"] = _targets(N, d, layout, X, g)
        st["loss"] = torch.empty(1, dtype=torch.float32, device=DEV)
    if case["deterministic"]:
        st["ws"] = torch.empty(tdmap.tdmap_workspace_size(op, N, d, 0, 0, 1), dtype=torch.uint8,
                               device=DEV)
    return st


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "edm":
        return tdmap.edm(state["X"], layout=c["layout"], out=state["out"])
    if kind == "cell":
        return tdmap.edm(state["X"], layout=c["layout"], rho=c["rho"], out=state["out"])
    if kind == "autograd":
        D = tdmap.EDM().apply(state["X"])
        (g,) = torch.autograd.grad(D, state["X"], state["dD"])
        return {"D": D.detach(), "dX": g}
    if kind == "backward":
        return tdmap.edm_backward(state["X"], state["dD"], layout=c["layout"],
                                  deterministic=c["deterministic"], out=state["dX"],
                                  workspace=state.get("ws"))
    if kind == "stress":
        loss, dX = tdmap.stress_backward(state["X"], state["delta"], layout=c["layout"],
                                         deterministic=c["deterministic"], out=state["dX"],
                                         loss=state["loss"], workspace=state.get("ws"))
        return {"loss": loss, "dX": dX}
    if kind == "gram":
        return tdmap.edm(state["X"], layout="packed", precision=c["precision"], out=state["out"],
                         workspace=state["ws"])
    return tdmap.edm_batched(state["X"], state["po"], state["oo"], out=state["out"],
                             workspace=state["ws"])


def work(case):
    """Each input read once, each output written once; per pair: d
    differences and d multiply-adds (Gram form: d multiply-adds, three times
    over in the split form), as much again and half for a gradient."""
    kind = case["kind"]
    d = case["d"]
    if kind == "batched":
        n, po, oo = _set_sizes(case)
        cells = int(oo[-1])
        return {"bytes": 4 * cells + 4 * d * int(po[-1]) + 16 * (case["sets"] + 1),
                "flops": cells * 3 * d}
    N = case["N"]
    pts = 4 * N * d
    if kind in ("edm", "cell"):
        cells = _cells(N, case["layout"])
        return {"bytes": 4 * cells + pts, "flops": cells * 3 * d}
    if kind == "gram":
        cells = _cells(N, "packed")
        mul = 3 if case["precision"] == "bf16x3_gram" else 1
        return {"bytes": 4 * cells + pts, "flops": cells * 2 * d * mul}
    if kind == "autograd":
        cells = _cells(N, "packed")
        return {"bytes": 8 * cells + 3 * pts, "flops": cells * 10 * d}
    cells = N * (N - 1) // 2
    return {"bytes": 4 * cells + 2 * pts, "flops": cells * 7 * d}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _dist(X, r0, r1):
    """Distances of rows r0 .. r1 - 1 to points 0 .. r1 - 1, difference form."""
    s = torch.zeros((r1 - r0, r1), dtype=X.dtype, device=X.device)
    for k in range(X.shape[1]):
        t = X[r0:r1, k, None] - X[None, :r1, k]
        s.addcmul_(t, t)
    return s.sqrt_()


def _dist_products(X, r0, r1):
    """The same through products (for wide points), the diagonal set to 0."""
    n = (X * X).sum(1)
    s = n[r0:r1, None] + n[None, :r1] - 2.0 * (X[r0:r1] @ X[:r1].t())
    s = s.clamp_min_(0.0).sqrt_()
    i = torch.arange(r0, r1, device=X.device)
    s[i - r0, i] = 0.0
    return s


def _unpack_rows(P, r0, r1, layout):
    """Rows r0 .. r1 - 1, columns 0 .. r1 - 1 of a buffer, zero on and above
    the diagonal."""
    if layout == "full":
        return torch.tril(P[r0:r1, :r1], diagonal=r0 - 1).double()
    strict = 1 if layout == "strict" else 0
    v = torch.zeros((r1 - r0, r1), dtype=torch.float32, device=P.device)
    keep = torch.ones_like(v, dtype=torch.bool).tril_(diagonal=r0 - strict)
    v[keep] = P[(_cells(r0, layout) if r0 else 0):_cells(r1, layout)]
    return torch.tril(v, diagonal=r0 - 1).double()


def _gradient(X, N, d, values):
    """dX from `values(r0, r1, D)` = dL/dD over rows r0 .. r1 - 1 (zero on and
    above the diagonal)."""
    dX = torch.zeros((N, d), dtype=torch.float64, device=DEV)
    step = _rows_per_block(N)
    for r0 in range(0, N, step):
        r1 = min(N, r0 + step)
        D = _dist(X, r0, r1)
        c = values(r0, r1, D)
        c = torch.where(D > 0, c / D, torch.zeros_like(c))
        for k in range(d):
            t = c * (X[r0:r1, k, None] - X[None, :r1, k])
            dX[r0:r1, k] += t.sum(1)
            dX[:r1, k] -= t.sum(0)
    return dX


def exact(case, seed):
    st = prepare(case, seed)
    kind = case["kind"]
    d = case["d"]
    X = st["X"].detach().double()
    if kind == "batched":
        _, po, oo = _set_sizes(case)
        st["out"] = None
        out = torch.empty(int(oo[-1]), dtype=torch.float64, device=DEV)
        for s in range(case["sets"]):
            if po[s + 1] > po[s]:
                Y = X[int(po[s]):int(po[s + 1])]
                n = Y.shape[0]
                out[int(oo[s]):int(oo[s + 1])] = _pack(lambda a, b: _dist(Y, a, b), n, "packed",
                                                       torch.float64)
        return out
    N = case["N"]
    if kind in ("edm", "cell"):
        st["out"] = None
        return _pack(lambda a, b: _dist(X, a, b), N, case["layout"], torch.float64)
    if kind == "gram":
        st["out"] = None
        return _pack(lambda a, b: _dist_products(X, a, b), N, "packed", torch.float64)
    if kind == "autograd":
        D = _pack(lambda a, b: _dist(X, a, b), N, "packed", torch.float64)
        return {"D": D, "dX": _gradient(X, N, d, lambda a, b, _: _unpack_rows(st["dD"], a, b,
                                                                              "packed"))}
    layout = case["layout"]
    if kind == "backward":
        return _gradient(X, N, d, lambda a, b, _: _unpack_rows(st["dD"], a, b, layout))
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)

    def residual(a, b, D):
        e = torch.tril(D, diagonal=a - 1) - _unpack_rows(st["delta"], a, b, layout)
        loss.add_(e.square().sum())
        return 2.0 * e

    dX = _gradient(X, N, d, residual)
    return {"loss": loss, "dX": dX}
