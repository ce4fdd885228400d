"""GPU parity of the graph preprocessing of Graph-SNMPBB (snmf_knn, snmf_knn_graph;
Section 2.2, eq. (2.3)) against the oracle (oracle/graph.py) on the same points.

Neighbour lists and the CSR pattern are integer results: they must be identical (both
sides rank by FP64 distance, ties to the lower index).  The values (Gaussian kernel,
normalised Laplacian) are FP64 on the device and rounded to the output type: within 1e-12
(F64) or 2^-24 plus one rounding (F32, bound 2e-7) of the entry, relative to max |entry|.
"""
import numpy as np
import pytest

import oracle as O
from paper_2606_02887_amd import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"
DT = {"f64": torch.float64, "f32": torch.float32}


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_02887_amd import snmf
    return snmf


def _points(n, dim, k, seed):
    rng = np.random.default_rng(seed)
    labels = np.repeat(np.arange(k), n // k + 1)[:n]
    return gen.cluster_features(labels, k, dim, rng)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,dim,K", [(3000, 16, 10), (997, 3, 1), (1500, 64, 40), (400, 7, 64)])
def test_knn_matches_oracle(S, prec, n, dim, K):
    X = torch.from_numpy(_points(n, dim, 8, n + dim)).to(DEV, DT[prec])
    nbr = S.knn(X, K).cpu().numpy()
    idx, _ = O.knn(X.double().cpu().numpy(), K)
    assert np.array_equal(nbr, idx)


def test_knn_ties_go_to_the_lower_index(S):
    """Integer points on a line: exact ties everywhere; neighbours i - 1, i + 1, i - 2, ..."""
    X = torch.arange(300, dtype=torch.float64, device=DEV)[:, None].contiguous()
    nbr = S.knn(X, 4).cpu().numpy()
    idx, _ = O.knn(X.cpu().numpy(), 4)
    assert np.array_equal(nbr, idx)
    assert list(nbr[10]) == [9, 11, 8, 12]


@pytest.mark.parametrize("n,dim,K", [(2, 1, 1), (2000, 3, 17), (2001, 1, 1), (2001, 4, 16),
                                     (2032, 5, 17), (2047, 8, 32), (2100, 9, 33), (2049, 16, 10),
                                     (2008, 17, 64), (2017, 32, 16), (2065, 33, 10), (2048, 48, 7),
                                     (2011, 64, 2)])
@pytest.mark.parametrize("kind", ["lattice", "equal", "tiny", "huge", "far"])
def test_knn_edges(S, n, dim, K, kind):
    """Identical lists at the edges of the tiles of points, of coordinates and of the lists,
    for data that screening by |x_j|^2 - 2 <x_i, x_j> cannot separate: exact ties, equal
    points, squares that underflow, squares near the overflow (distances below it) and
    a cloud far from the origin."""
    rng = np.random.default_rng(n * 64 + dim)
    X = rng.integers(0, 3, (n, dim)).astype(np.float64)
    X = {"lattice": X, "equal": np.ones((n, dim)), "tiny": X * 1e-161,
         "huge": 1e153 * (1 + 0.01 * rng.random((n, dim))),
         "far": 1e6 + rng.random((n, dim))}[kind]
    nbr = S.knn(torch.from_numpy(X).to(DEV), K).cpu().numpy()
    if kind == "tiny":  # the rounding of the sums of underflowed squares: order of addition
        d = np.zeros((n, n))
        for c in range(dim):
            t = X[:, c][:, None] - X[:, c][None, :]
            d = d + t * t
        got = np.take_along_axis(d, nbr, 1)
        d[np.arange(n), np.arange(n)] = np.inf
        ref = np.sort(d, 1)[:, :K]
        assert np.abs(got - ref).max() <= dim * 2.0 ** -1074
    else:
        idx, _ = O.knn(X, K)
        assert np.array_equal(nbr, idx)


@pytest.mark.parametrize("n,dim,K", [(2001, 32, 17), (2401, 3, 3), (2402, 5, 10), (2601, 9, 20),
                                     (2617, 17, 17), (3001, 16, 16), (2003, 33, 11), (2049, 4, 64),
                                     (2003, 33, 33), (2100, 64, 40), (2064, 48, 5)])
@pytest.mark.parametrize("kind", ["lattice", "thirds", "equal", "far", "spread"])
def test_knn_edges_fp32(S, n, dim, K, kind):
    """As above in FP32, just past the sizes from which the search is screened: every width of
    the coordinates' blocks, both forms of their loads, one and two sets of first limits;
    data that the screen separates (spread), that pass it in part (lattice, thirds: three
    points many times over) and that it hands to the search without a screen."""
    rng = np.random.default_rng(n * 64 + dim)
    X = {"lattice": rng.integers(0, 3, (n, dim)).astype(np.float64),
         "thirds": rng.standard_normal((3, dim))[np.arange(n) % 3],
         "equal": np.full((n, dim), 0.3), "far": 1e6 + rng.random((n, dim)),
         "spread": rng.standard_normal((n, dim))}[kind]
    X = torch.from_numpy(X).to(DEV, torch.float32)
    idx, _ = O.knn(X.double().cpu().numpy(), K)
    assert np.array_equal(S.knn(X, K).cpu().numpy(), idx)


@pytest.mark.parametrize("n,dim,K", [(300, 3, 7), (2500, 16, 10), (2500, 9, 5), (2100, 32, 40)])
@pytest.mark.parametrize("part", [1, 3])
def test_knn_distances_beyond_the_largest_double(S, n, dim, K, part):
    """Finite FP64 points whose squared distances overflow (all of them, or a third): the lists
    still hold K other points, those at overflowing distances by index, and the graph is
    that of the lists."""
    rng = np.random.default_rng(n + dim)
    X = rng.standard_normal((n, dim))
    X[::part] *= 1e200
    X[5] = X[8]                           # a distance of zero among them
    Xt = torch.from_numpy(X).to(DEV)
    nbr = S.knn(Xt, K).cpu().numpy()
    for i in np.unique(np.r_[0:20, rng.integers(0, n, 40), n - 1]):
        with np.errstate(over="ignore"):
            d = np.sum((X - X[i]) ** 2, axis=1)
        order = np.lexsort((np.arange(n), d))
        assert np.array_equal(nbr[i], order[order != i][:K]), i
    rowptr, col, _ = (t.cpu().numpy() for t in S.knn_graph(Xt, K, laplacian=False).keep)
    pairs = np.repeat(np.arange(n), K) * n + nbr.reshape(-1)
    both = np.unique(np.r_[pairs, pairs % n * n + pairs // n])
    assert np.array_equal(np.repeat(np.arange(n), np.diff(rowptr)) * n + col, both)


def test_knn_graph_long_rows(S):
    """A star: the hub's row of the union holds every point (the sort of rows past 64)."""
    n = 700
    X = np.zeros((n, 64))
    rng = np.random.default_rng(9)
    X[1:] = rng.standard_normal((n - 1, X.shape[1]))
    X[1:] /= np.linalg.norm(X[1:], axis=1)[:, None]   # all closer to 0 than to each other
    M = S.knn_graph(torch.from_numpy(X).to(DEV), 2, laplacian=False)
    rowptr, col, _ = (t.cpu().numpy() for t in M.keep)
    ref = O.similarity(X, 2, 0.0)
    assert np.array_equal(rowptr, ref.indptr) and np.array_equal(col, ref.indices)
    assert rowptr[1] - rowptr[0] > 128


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("laplacian,sigma", [(True, 0.0), (False, 0.0), (True, 1.5), (False, 2.0)])
def test_knn_graph_matches_oracle(S, prec, laplacian, sigma):
    n, dim, K = 2500, 16, 10
    X = torch.from_numpy(_points(n, dim, 10, 5)).to(DEV, DT[prec])
    M = S.knn_graph(X, K, sigma=sigma, laplacian=laplacian)
    rowptr, col, val = (t.cpu().numpy() for t in M.keep)
    Xo = X.double().cpu().numpy()
    ref = O.knn_laplacian(Xo, K, sigma) if laplacian else O.similarity(Xo, K, sigma)
    assert np.array_equal(rowptr, ref.indptr) and np.array_equal(col, ref.indices)
    err = np.abs(val.astype(np.float64) - ref.data).max() / np.abs(ref.data).max()
    assert err <= (1e-12 if prec == "f64" else 2e-7), err


def test_graph_solve_on_the_device_laplacian(S):
    """Graph-SNMPBB with the Laplacian built on the device: the same solve as with the
    oracle's Laplacian (identical pattern, values to FP32 rounding), 30 outer iterations
    in FP64 from the same start, residual and projected-gradient norm to 1e-9."""
    p = gen.sbm_problem(n=1200, k=6, r=6, p_in=0.06, p_out=0.003, seed=41)
    A = p["A"]
    Xt = torch.from_numpy(p["X"]).to(DEV, torch.float64)
    Lg = S.knn_graph(Xt, p["knn"])
    Lo = O.knn_laplacian(p["X"], p["knn"])
    lam = O.default_lambda(A)
    W, Ht, info = S.solve(S.csr_from_scipy(A, torch.float64),
                          torch.from_numpy(p["W0"]).to(DEV, torch.float64),
                          S.params(lam=lam, gamma=0.2, prec=S.F64, max_outer=30), Lg)
    _, _, hist = O.snmpbb(A, p["W0"], O.Params(lam=lam, gamma=0.2), 30, L=Lo)
    assert abs(info["res_WH"] - hist[-1]["res_WH"]) <= 1e-9 * hist[-1]["res_WH"]
    assert abs(info["pg_norm"] - hist[-1]["pg"]) <= 1e-9 * hist[-1]["pg"]


def test_graph_error_codes(S):
    X = torch.rand((50, 4), dtype=torch.float32, device=DEV)
    bad = X.clone()
    bad[7, 2] = float("nan")
    with pytest.raises(S.SnmfError) as e:
        S.knn(bad, 3)
    assert e.value.name == "E_NONFINITE"
    with pytest.raises(S.SnmfError) as e:
        S.knn(X, 50)
    assert e.value.name == "E_SHAPE"
    with pytest.raises(S.SnmfError) as e:
        S.knn_graph(torch.rand((50, 65), dtype=torch.float32, device=DEV), 3)
    assert e.value.name == "E_SHAPE"
