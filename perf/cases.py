"""Timing cases: one pass each through the public entry points of paper_2606_02887_amd.snmf,
on inputs made from a seed on the GPU (no scipy, so that many of them can be made quickly).

The kinds follow the framework's uses:

* solve -- SNMPBB on one matrix (dense, Laplacian-regularised graph, or low-rank surrogate).
  A program keeps the plan (scratch, input checks, the BF16 split) and solves from starts; the
  one-shot form creates and drops the plan inside the call.
* batch -- many graphs and restarts solved together through one kept batch.
* nmf -- rectangular NMF in one call (the library transposes V inside it).
* sketch -- the range finder that builds the low-rank surrogate of a sparse graph.
* knn -- the K-nearest-neighbour Laplacian of a point set.
* train -- steps of the warm-start network's training on a kept row pool.

Solves run a handful of outer iterations: the iteration amplifies rounding-size differences
(a thousandfold within some tens of iterations in single precision), so factors after
hundreds of iterations of two correct programs need not agree, while the work of an outer
iteration does not depend on how many there are.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_02887_amd import snmf as S

DEV = "cuda"
PREC = {"f64": S.F64, "f32": S.F32, "bf16x3": S.BF16X3}
DTYPE = {"f64": torch.float64, "f32": torch.float32, "bf16x3": torch.float32}
INNER = 5                      # inner iterations of a half-step (the library's default)


# --------------------------------------------------------------------------- the cases
def listed():
    return [
        # a row of the paper's synthetic table: a call of a few microseconds per kernel, where
        # only latency and the number of launches count; double precision as in MATLAB
        {"name": "dense_f64_small", "kind": "solve", "fmt": "dense", "prec": "f64", "n": 200,
         "r": 5, "outer": 10, "oneshot": False},
        # the table's largest row as one call: plan, input checks and solve together
        {"name": "dense_f64_oneshot", "kind": "solve", "fmt": "dense", "prec": "f64", "n": 1000,
         "r": 20, "outer": 10, "oneshot": True},
        # an ordinary dense problem of no particular size: odd n, odd rank
        {"name": "dense_f32_ragged", "kind": "solve", "fmt": "dense", "prec": "f32", "n": 3001,
         "r": 21, "outer": 4, "oneshot": False},
        # the headline problem in both of its precisions
        {"name": "dense_f32_headline", "kind": "solve", "fmt": "dense", "prec": "f32", "n": 8192,
         "r": 64, "outer": 4, "oneshot": False},
        {"name": "dense_bf16x3_headline", "kind": "solve", "fmt": "dense", "prec": "bf16x3",
         "n": 8192, "r": 64, "outer": 4, "oneshot": False},
        # clustering a graph with the Laplacian regulariser
        {"name": "graph_laplacian", "kind": "solve", "fmt": "graph", "prec": "f32", "n": 20000,
         "r": 20, "outer": 8, "oneshot": False},
        # the low-rank surrogate of a large graph
        {"name": "lowrank_large", "kind": "solve", "fmt": "lowrank", "prec": "f32", "n": 200000,
         "r": 32, "ell": 64, "outer": 4, "oneshot": False},
        # many small graphs with restarts in one batch
        {"name": "batch_graphs", "kind": "batch", "prec": "f32", "graphs": 30, "n_lo": 500,
         "n_hi": 5000, "restarts": 8, "outer": 4},
        # rectangular NMF, the dense benchmark size
        {"name": "nmf_dense", "kind": "nmf", "prec": "f32", "m": 8192, "n": 4096, "r": 64,
         "outer": 4},
        # the range finder on a power-law graph: 64 + 10 columns, two power iterations
        {"name": "sketch_powerlaw", "kind": "sketch", "prec": "f32", "n": 200000, "rank": 64,
         "over": 10, "power": 2, "degree": 10},
        # the graph workload's preprocessing
        {"name": "knn_laplacian", "kind": "knn", "prec": "f32", "n": 20000, "dim": 16, "K": 10,
         "sigma": 0.0},
        # training steps of the warm-start network at its minibatch size
        {"name": "train_network", "kind": "train", "r": 16, "batch": 4096, "pool": 200000,
         "steps": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "solve", "batch", "nmf", "sketch",
                       "knn", "train"])
    if kind == "solve":
        fmt = rng.choice(["dense", "dense", "dense", "graph", "lowrank"])
        if fmt == "dense":
            prec = rng.choice(["f64", "f32", "f32", "bf16x3"])
            n = _log(rng, 100, 2500) if prec == "f64" else _log(rng, 500, 8192)
            return {"kind": kind, "fmt": fmt, "prec": prec, "n": n,
                    "r": _log(rng, 2, 24 if prec == "f64" else 64),
                    "outer": rng.randint(4, 10) if prec == "f64" else rng.randint(3, 4),
                    "oneshot": rng.random() < 0.25}
        if fmt == "graph":
            return {"kind": kind, "fmt": fmt, "prec": "f32", "n": _log(rng, 2000, 20000),
                    "r": rng.randint(5, 24), "outer": rng.randint(4, 8), "oneshot": False}
        return {"kind": kind, "fmt": fmt, "prec": "f32", "n": _log(rng, 10000, 200000),
                "r": rng.randint(5, 32), "ell": rng.randint(40, 64), "outer": rng.randint(3, 4),
                "oneshot": False}
    if kind == "batch":
        return {"kind": kind, "prec": "f32", "graphs": rng.randint(8, 30), "n_lo": 300,
                "n_hi": rng.randint(1000, 4000), "restarts": rng.randint(1, 8), "outer": 4}
    if kind == "nmf":
        return {"kind": kind, "prec": "f32", "m": _log(rng, 1000, 8192),
                "n": _log(rng, 500, 4096), "r": rng.randint(8, 64), "outer": rng.randint(3, 4)}
    if kind == "sketch":
        return {"kind": kind, "prec": rng.choice(["f32", "f64"]), "n": _log(rng, 20000, 200000),
                "rank": rng.randint(16, 64), "over": rng.randint(5, 10), "power": rng.randint(1, 2),
                "degree": rng.randint(6, 10)}
    if kind == "knn":
        return {"kind": kind, "prec": rng.choice(["f32", "f64"]), "n": _log(rng, 2000, 20000),
                "dim": rng.randint(3, 16), "K": rng.randint(5, 16),
                "sigma": rng.choice([0.0, 2.0])}
    return {"kind": kind, "r": rng.choice([8, 16, 32]), "batch": _log(rng, 512, 4096),
            "pool": _log(rng, 20000, 200000), "steps": rng.randint(4, 8)}


# --------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(g, *shape, dtype=torch.float64):
    return torch.rand(shape, generator=g, device=DEV, dtype=dtype)


def _randn(g, *shape, dtype=torch.float64):
    return torch.randn(shape, generator=g, device=DEV, dtype=dtype)


def _csr_of_keys(key, val, n):
    """CSR arrays (rowptr int64, col int32, val) from sorted keys row * n + col."""
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0)
    return rowptr, (key % n).to(torch.int32).contiguous(), val.contiguous()


def _factor(g, n, r, uniform):
    """A planted factor: uniform entries (the paper's synthetic problems), or overlapping
    communities -- every row belongs to one column strongly and to each other one with
    probability 0.1 (what a clustering or topic problem looks like)."""
    w = _rand(g, n, r)
    if uniform:
        return w
    w *= _rand(g, n, r) < 0.1
    own = torch.randint(0, r, (n,), generator=g, device=DEV)
    w[torch.arange(n, device=DEV), own] += 0.5 + _rand(g, n)
    return w


def _planted(g, m, n, r, symmetric, uniform):
    """max(W* H*^T + E, 0), the Gaussian noise E with 1% of the mean entry."""
    w = _factor(g, m, r, uniform)
    h = w if symmetric else _factor(g, n, r, uniform)
    a = w @ h.T
    a += (0.01 * float(a.mean())) * _randn(g, m, n)
    if symmetric:
        a = torch.triu(a)
        a = a + torch.triu(a, 1).T
    return torch.clamp_(a, min=0.0)


def _sbm(g, n, k, p_in=0.02, p_out=0.0005):
    """Normalised adjacency D^-1/2 Adj D^-1/2 of a stochastic block model with k equal
    clusters, and its labels."""
    labels = torch.arange(n, device=DEV) * k // n
    u = _rand(g, n, n, dtype=torch.float32)
    hit = u < torch.where(labels[:, None] == labels[None, :], p_in, p_out)
    hit = torch.triu(hit, 1)
    hit |= hit.T.clone()
    idx = torch.nonzero(hit)
    key = idx[:, 0] * n + idx[:, 1]
    d = torch.bincount(idx[:, 0], minlength=n).double()
    s = torch.where(d > 0, d.clamp(min=1.0).rsqrt(), torch.zeros_like(d))
    return _csr_of_keys(key, s[idx[:, 0]] * s[idx[:, 1]], n), labels


def _features(g, labels, k, dim):
    mu = 2.0 * _randn(g, k, dim)
    return mu[labels] + _randn(g, labels.numel(), dim)


def _laplacian(g, labels, k, K):
    """I - D^-1/2 V D^-1/2 of an unweighted neighbour graph (union pattern): every node lists
    K random nodes of its own cluster, as separated clusters of features give."""
    n = labels.numel()
    row = torch.arange(n, device=DEV)[:, None].expand(n, K).reshape(-1)
    lo, hi = -(-labels * n // k), -(-(labels + 1) * n // k)     # a cluster's contiguous rows
    col = (lo[row] + (_rand(g, n * K) * (hi - lo)[row]).long()).clamp(max=n - 1)
    row, col = row[row != col], col[row != col]
    edge = torch.unique(torch.cat([row * n + col, col * n + row]))
    deg = torch.bincount(edge // n, minlength=n).double()
    key = torch.cat([edge, torch.arange(n, device=DEV) * (n + 1)])
    val = torch.cat([-(deg[edge // n] * deg[edge % n]).rsqrt(),
                     torch.ones(n, dtype=torch.float64, device=DEV)])
    key, order = torch.sort(key)
    return _csr_of_keys(key, val[order], n)


def _powerlaw(g, n, degree):
    """Symmetric power-law graph (exponent 2.1), mean degree about `degree`, values in (0, 1]."""
    cap = math.sqrt(n * degree)
    d = torch.floor((0.1 * degree) * (1.0 - _rand(g, n)).pow(-1.0 / 1.1)).clamp(1, cap)
    row = torch.repeat_interleave(torch.arange(n, device=DEV), d.long())
    col = torch.searchsorted(torch.cumsum(d, 0), _rand(g, row.numel()) * d.sum()).clamp(max=n - 1)
    keep = row != col
    row, col = row[keep], col[keep]
    pair = torch.unique(torch.minimum(row, col) * n + torch.maximum(row, col))
    v = 1.0 - _rand(g, pair.numel())
    lo, hi = pair // n, pair % n
    key, order = torch.sort(torch.cat([lo * n + hi, hi * n + lo]))
    return _csr_of_keys(key, torch.cat([v, v])[order], n)


def _lowrank(g, n, ell):
    """(U, lam), U lam U^T = W* W*^T for a factor of ell overlapping communities of unequal
    weight: the exact eigenpairs of a low-rank nonnegative matrix; and its mean entry."""
    w = _factor(g, n, ell, False)
    w *= torch.linspace(1.0, 0.3, ell, dtype=torch.float64, device=DEV)
    e, p = torch.linalg.eigh(w.T @ w)
    return (w @ p) / e.sqrt(), e, float((w.sum(0) ** 2).sum()) / n / n


def _start(g, n, r, mean):
    return _rand(g, n, r) * math.sqrt(mean / r)


def _as(x, dtype):
    return x.to(dtype).contiguous()


def _inputs(case, seed):
    """The arrays of a case in their stored types."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "solve":
        dt, n, r = DTYPE[case["prec"]], case["n"], case["r"]
        if case["fmt"] == "dense":
            a = _planted(g, n, n, r, True, case["prec"] == "f64")
            return {"A": _as(a, dt), "W0": _as(_start(g, n, r, float(a.mean())), dt),
                    "lam": 0.01 * float(a.norm())}
        if case["fmt"] == "graph":
            a, labels = _sbm(g, n, r, 0.02 * 20000 / n * r / 20, 0.0005 * 20000 / n)
            L = _laplacian(g, labels, r, 10)
            return {"A": (a[0], a[1], _as(a[2], dt)), "L": (L[0], L[1], _as(L[2], dt)),
                    "W0": _as(_start(g, n, r, float(a[2].sum()) / n / n), dt),
                    "lam": 0.01 * float(a[2].norm())}
        U, e, mean = _lowrank(g, n, case["ell"])
        return {"U": _as(U, dt), "E": e.contiguous(), "W0": _as(_start(g, n, r, mean), dt),
                "lam": 0.01 * float(e.norm())}
    if kind == "batch":
        dt, out = DTYPE[case["prec"]], []
        host = np.random.default_rng(case["graphs"])      # the sizes belong to the case
        for _ in range(case["graphs"]):
            n = int(host.integers(case["n_lo"], case["n_hi"] + 1))
            r = int(host.choice([8, 16, 32]))
            a, _ = _sbm(g, n, r, min(0.9, 30.0 * r / n), 4.0 / n)
            w0 = _rand(g, case["restarts"], n, r) * math.sqrt(float(a[2].sum()) / n / n / r)
            out.append({"A": (a[0], a[1], _as(a[2], dt)), "n": n, "r": r, "W0": _as(w0, dt),
                        "lam": 0.01 * float(a[2].norm())})
        return {"graphs": out}
    if kind == "nmf":
        dt, m, n, r = DTYPE[case["prec"]], case["m"], case["n"], case["r"]
        v = _planted(g, m, n, r, False, False)
        mean = float(v.mean())
        return {"V": _as(v, dt), "W0": _as(_start(g, m, r, mean), dt),
                "Ht0": _as(_start(g, n, r, mean), dt)}
    if kind == "sketch":
        dt = DTYPE[case["prec"]]
        a = _powerlaw(g, case["n"], case["degree"])
        return {"A": (a[0], a[1], _as(a[2], dt)),
                "Omega": _as(_randn(g, case["n"], case["rank"] + case["over"]), dt)}
    if kind == "knn":
        labels = torch.arange(case["n"], device=DEV) * 20 // case["n"]
        return {"X": _as(_features(g, labels, 20, case["dim"]), DTYPE[case["prec"]])}
    # train: a network some hundred steps into its training (nonzero second layer and moments)
    r, h = case["r"], 128
    host = np.random.default_rng(seed)
    init = {"M1": host.standard_normal((h, r)) * math.sqrt(2.0 / r),
            "b1": 0.1 * host.standard_normal(h), "M2": 0.1 * host.standard_normal((r, h)),
            "b2": 0.05 * host.standard_normal(r)}
    npar = 2 * h * r + h + r
    C = _randn(g, case["pool"], r, dtype=torch.float32)
    T = torch.clamp(C + 0.5 * _randn(g, case["pool"], r, dtype=torch.float32), min=0.0)
    idx = torch.randint(0, case["pool"], (case["steps"], case["batch"]), generator=g, device=DEV)
    return {"init": init, "C": C, "T": T, "idx": idx.to(torch.int32),
            "m": 1e-3 * _randn(g, npar, dtype=torch.float32),
            "v": 1e-5 * (0.5 + _rand(g, npar, dtype=torch.float32))}


def prepare(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    st = {"case": case}
    if kind == "solve":
        prm = S.params(lam=x["lam"], gamma=0.2 if case["fmt"] == "graph" else 0.0,
                       prec=PREC[case["prec"]], max_outer=case["outer"], check_every=1 << 30)
        L = None
        if case["fmt"] == "dense":
            A = S.dense(x["A"])
        elif case["fmt"] == "graph":
            A, L = S.csr(*x["A"], case["n"]), S.csr(*x["L"], case["n"])
        else:
            A = S.lowrank(x["U"], x["E"])
        st.update(A=A, W0=x["W0"], prm=prm)
        if not case["oneshot"]:
            st["plan"] = S.Plan(A, case["r"], prm, L)
    elif kind == "batch":
        gs = x["graphs"]
        prm = S.params(prec=PREC[case["prec"]], max_outer=case["outer"], check_every=1 << 30)
        st["batch"] = S.Batch([S.csr(*q["A"], q["n"]) for q in gs], [q["r"] for q in gs], prm,
                              case["restarts"], lam=[q["lam"] for q in gs])
        st["W0s"] = [q["W0"] for q in gs]
    elif kind == "nmf":
        st.update(V=S.dense(x["V"]), W0=x["W0"], Ht0=x["Ht0"],
                  prm=S.params(lam=0.0, prec=PREC[case["prec"]], max_outer=case["outer"],
                               check_every=1 << 30))
    elif kind == "sketch":
        st.update(A=S.csr(*x["A"], case["n"]), Omega=x["Omega"])
    elif kind == "knn":
        st["X"] = x["X"]
    else:
        net = S.Mlp(x["init"])
        net.adam_m.copy_(x["m"])
        net.adam_v.copy_(x["v"])
        net.step = 300
        st.update(net=net, C=x["C"], T=x["T"], idx=x["idx"])
    return st


# --------------------------------------------------------------------------- one pass
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "solve":
        if case["oneshot"]:
            W, Ht, info = S.solve(st["A"], st["W0"], st["prm"], trace=False)
        else:
            W, Ht, info = st["plan"].solve(st["W0"], trace=False)
        return {"W": W, "Ht": Ht, "res": info["res_WH"]}
    if kind == "batch":
        Ws, Hs, infos, _ = st["batch"].solve(st["W0s"])
        return {"W": Ws, "Ht": Hs,
                "res": np.array([q["res_WH"] for q in infos], dtype=np.float32)}
    if kind == "nmf":
        W, Ht, info = S.nmf_solve(st["V"], case["n"], st["W0"], st["Ht0"], st["prm"], trace=False)
        return {"W": W, "Ht": Ht, "res": info["res_WH"]}
    if kind == "sketch":
        U, lam = S.lai_sketch(st["A"], case["rank"], case["power"], st["Omega"])
        return {"U": U, "lam": lam}
    if kind == "knn":
        rowptr, col, val = S.knn_graph(st["X"], case["K"], sigma=case["sigma"]).keep
        tail = (0, case["n"] * (2 * case["K"] + 1) - col.numel())     # one shape for any points
        return {"rowptr": rowptr, "col": torch.nn.functional.pad(col, tail),
                "val": torch.nn.functional.pad(val, tail)}
    net = st["net"]
    for q in range(case["steps"]):
        net.train_step(st["C"], st["T"], st["idx"][q], 1.0, 1e-3)
    return {"M1": net.M1, "b1": net.b1, "M2": net.M2, "b2": net.b2}


# --------------------------------------------------------------------------- work
def _half_bytes(n, r, e):
    """An inner iteration cannot do without reading X, g and the partner's Gram and writing
    X, g; the gradient is formed once from the product, X and P."""
    return e * n * r * (4 * INNER + 5)


def _half_flops(n, r):
    return 2.0 * n * r * r * (1 + 3 * INNER)      # the Gram, then X G, Z G and D G


def work(case):
    kind = case["kind"]
    if kind == "solve":
        n, r, k = case["n"], case["r"], case["outer"]
        e = 8 if case["prec"] == "f64" else 4
        if case["fmt"] == "dense":
            prod_b, prod_f = e * n * n + 2 * e * n * r, 2.0 * n * n * r
            if case["prec"] == "bf16x3":
                prod_f *= 3
            once = e * n * n if case["oneshot"] else 0
        elif case["fmt"] == "graph":
            nnz = 30 * n
            prod_b, prod_f = 8 * nnz + 8 * n + 2 * e * n * r, 2.0 * nnz * r
            lap = 12 * n                                      # L X, L Z, L D, L S of the H-step
            prod_b += (1 + 3 * INNER) / 2 * (8 * lap + 8 * n + 2 * e * n * r)
            prod_f += (1 + 3 * INNER) / 2 * 2.0 * lap * r
            once = 0
        else:
            ell = case["ell"]
            prod_b, prod_f = 2 * e * n * ell + 2 * e * n * r, 4.0 * n * ell * r
            once = 0
        return {"bytes": once + 2 * k * (prod_b + _half_bytes(n, r, e)),
                "flops": 2 * k * (prod_f + _half_flops(n, r))}
    if kind == "batch":
        n, r, k = 0.5 * (case["n_lo"] + case["n_hi"]), 56.0 / 3, case["outer"]
        inst = case["graphs"] * case["restarts"]
        deg = 30.0
        return {"bytes": 2 * k * (case["graphs"] * 8 * deg * n
                                  + inst * (8 * n * r + _half_bytes(n, r, 4))),
                "flops": 2 * k * inst * (2.0 * deg * n * r + _half_flops(n, r))}
    if kind == "nmf":
        m, n, r, k = case["m"], case["n"], case["r"], case["outer"]
        return {"bytes": 4 * m * n + k * (8 * m * n + 8 * (m + n) * r
                                          + _half_bytes(m, r, 4) + _half_bytes(n, r, 4)),
                "flops": k * (4.0 * m * n * r + _half_flops(m, r) + _half_flops(n, r))}
    if kind == "sketch":
        n, w, q = case["n"], case["rank"] + case["over"], case["power"]
        e = 8 if case["prec"] == "f64" else 4
        nnz = case["degree"] * n
        return {"bytes": (2 * q + 2) * ((4 + e) * nnz + 2 * e * n * w)
                + (2 * q + 1) * 2 * e * n * w + e * n * (w + case["rank"]),
                "flops": (2 * q + 2) * 2.0 * nnz * w + (2 * q + 1) * 4.0 * n * w * w}
    if kind == "knn":
        n, d, K = case["n"], case["dim"], case["K"]
        e = 8 if case["prec"] == "f64" else 4
        return {"bytes": e * n * d + 2 * K * n * (4 + e) + 8 * n, "flops": 3.0 * n * n * d}
    r, b, k = case["r"], case["batch"], case["steps"]
    return {"bytes": k * (8 * b * r + 4 * b + 24 * (256 * r + 128 + r)),
            "flops": k * 3 * 4.0 * b * 128 * r}


# --------------------------------------------------------------------------- 64 bits
def _inner(apply, X, P, lam, gamma=0.0, L=None):
    """Algorithm 1 on f(X) with the partner P fixed, INNER iterations: the projected
    Barzilai-Borwein method with a nonmonotone line search, objective differences in
    closed form (f is quadratic)."""
    G = P.T @ P
    rho = float(torch.linalg.eigvalsh(G)[-1])

    def hess(V):
        out = V @ G + lam * V
        return out + gamma * (L @ V) if L is not None else out

    g = X @ G - apply(P) + (lam * (X - P) if lam else 0.0)
    if L is not None:
        g = g + gamma * (L @ X)
    e, alpha, ss, sy = 0.0, 1.0 / rho, None, None
    for k in range(INNER):
        dZ = torch.clamp(X - g / rho, min=0.0) - X
        Z = X + dZ
        h = hess(dZ)
        gZ = g + h
        fZ = float((g * dZ).sum() + 0.5 * (dZ * h).sum())
        if k:
            alpha = min(1e10, max(1e-10, ss / sy if sy > 0 else 1e10))
        D = torch.clamp(Z - alpha * gZ, min=0.0) - Z
        delta, q = float((gZ * D).sum()), float((D * hess(D)).sum())
        beta, t = 1.0, 0
        while fZ + beta * delta + 0.5 * beta * beta * q > e + 1e-3 * beta * delta and t < 20:
            beta, t = 0.5 * beta, t + 1
        Xn = torch.clamp(Z + 1.7 * beta * D, min=0.0)
        Sk = Xn - X
        h = hess(Sk)
        ss, sy = float((Sk * Sk).sum()), float((Sk * h).sum())
        e = 0.85 * (e - float((g * Sk).sum()) - 0.5 * sy)
        X, g = Xn, g + h
        if ss == 0.0:
            break
    return X


def _solve64(apply, W0, lam, outer, normA2, gamma=0.0, L=None):
    W = W0.double()
    H = W.clone()
    for _ in range(outer):
        W = _inner(apply, W, H, lam)
        H = _inner(apply, H, W, lam, gamma, L)
    res2 = normA2 - 2.0 * float((apply(H) * W).sum()) + float(((W.T @ W) * (H.T @ H)).sum())
    return W, H, math.sqrt(max(res2, 0.0) / normA2)


def _sparse(a, n):
    return torch.sparse_csr_tensor(a[0], a[1].long(), a[2].double(), (n, n))


def _bf16(x):
    return x.to(torch.bfloat16).double()


def exact(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    if kind == "solve":
        k, lam = case["outer"], x["lam"]
        if case["fmt"] == "dense":
            A = x["A"].double()
            W, H, res = _solve64(lambda P: A @ P, x["W0"], lam, k, float((A * A).sum()))
        elif case["fmt"] == "graph":
            A, L = _sparse(x["A"], case["n"]), _sparse(x["L"], case["n"])
            W, H, res = _solve64(lambda P: A @ P, x["W0"], lam, k,
                                 float(x["A"][2].double().square().sum()), 0.2, L)
        else:
            U, e = x["U"].double(), x["E"]
            W, H, res = _solve64(lambda P: U @ (e[:, None] * (U.T @ P)), x["W0"], lam, k,
                                 float((e * e).sum()))
        return {"W": W, "Ht": H, "res": res}
    if kind == "batch":
        Ws, Hs = [], []
        for q in x["graphs"]:
            A = _sparse(q["A"], q["n"])
            nA2 = float(q["A"][2].double().square().sum())
            got = [_solve64(lambda P: A @ P, w, q["lam"], case["outer"], nA2) for w in q["W0"]]
            Ws.append(torch.stack([w for w, _, _ in got]))
            Hs.append(torch.stack([h for _, h, _ in got]))
        return {"W": Ws, "Ht": Hs, "res": None}
    if kind == "nmf":
        V = x["V"].double()
        W, H = x["W0"].double(), x["Ht0"].double()
        for _ in range(case["outer"]):
            W = _inner(lambda P: V @ P, W, H, 0.0)
            H = _inner(lambda P: V.T @ P, H, W, 0.0)
        return {"W": W, "Ht": H, "res": float((V - W @ H.T).norm() / V.norm())}
    if kind == "sketch":
        A = _sparse(x["A"], case["n"])
        Q = torch.linalg.qr(A @ x["Omega"].double()).Q
        for _ in range(2 * case["power"]):
            Q = torch.linalg.qr(A @ Q).Q
        e = torch.linalg.eigvalsh(Q.T @ (A @ Q))
        order = torch.argsort(e.abs(), descending=True)[: case["rank"]]
        return {"U": None, "lam": e[order]}        # the eigenvectors' signs are the method's own
    if kind == "knn":
        return None                                # whole numbers, and values pinned by them
    r, b = case["r"], case["batch"]
    M1, b1 = (torch.from_numpy(np.float32(x["init"][k])).to(DEV).double() for k in ("M1", "b1"))
    M2, b2 = (torch.from_numpy(np.float32(x["init"][k])).to(DEV).double() for k in ("M2", "b2"))
    par, m, v = [M1, b1, M2, b2], x["m"].double(), x["v"].double()
    sizes = [p.numel() for p in par]
    for q in range(case["steps"]):
        at = x["idx"][q].long()
        c, t = x["C"][at].double(), x["T"][at].double()
        q1, q2 = _bf16(par[0]), _bf16(par[2])
        z = c @ q1.T + par[1]
        a = torch.clamp(z, min=0.0)
        o = c + a @ q2.T + par[3]
        y = torch.clamp(o, min=0.0)
        gap = (y * y).mean() - (t * t).mean()
        do = (2.0 * (y - t) + 4.0 * gap * y) / (b * r) * (o > 0)
        da = (do @ q2) * (z > 0)
        grad = torch.cat([(da.T @ c).reshape(-1), da.sum(0), (do.T @ a).reshape(-1), do.sum(0)])
        step = 301 + q
        m = 0.9 * m + 0.1 * grad
        v = 0.999 * v + 0.001 * grad * grad
        upd = 1e-3 * (m / (1 - 0.9 ** step)) / ((v / (1 - 0.999 ** step)).sqrt() + 1e-8)
        par = [p - u.view_as(p) for p, u in zip(par, torch.split(upd, sizes))]
    return {"M1": par[0], "b1": par[1], "M2": par[2], "b2": par[3]}
