"""Per-kernel parity of the HIP primitives against the FP64 oracle on identical inputs.

Tolerances: normwise relative error <= 1e-12 (FP64 kernels; 1e-13 where the operation
is a single reduction), <= 1e-5 (FP32), BF16 split bit-exact against a round-to-nearest-
even emulation, split-BF16 product stated per case (<= 2e-5).
"""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle as O
from paper_2606_02887_amd import gen
from parity_util import comp_rel, nrel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_02887_amd import snmf
    return snmf


DEV = "cuda"


def _t(x, dtype):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV, dtype)


# ------------------------------------------------------------------ rho = ||G||_2
@pytest.mark.parametrize("r", [1, 2, 5, 10, 20, 31, 32, 33, 64])
def test_rho_matches_eigvalsh(S, r):
    rng = np.random.default_rng(r)
    P = rng.random((3 * r + 5, r))
    G = P.T @ P
    got = S.rho(_t(G, torch.float64))
    ref = O.spectral_norm_psd(G)
    assert abs(got - ref) <= 1e-13 * ref


def test_rho_near_degenerate_spectrum(S):
    """Equal-size clusters give G ~ c I: r nearly equal eigenvalues, still exact to 1e-13."""
    rng = np.random.default_rng(3)
    r, n = 20, 400
    P = 1e-8 * rng.random((n, r))
    P[np.arange(n), np.arange(n) % r] += 1.0 + 1e-6 * rng.random(n)
    G = P.T @ P
    ev = np.linalg.eigvalsh(G)
    assert (ev[-1] - ev[0]) / ev[-1] < 1e-5
    got = S.rho(_t(G, torch.float64))
    ref = O.spectral_norm_psd(G)
    assert abs(got - ref) <= 1e-13 * ref


@pytest.mark.parametrize("r", [2, 3, 21, 64])
@pytest.mark.parametrize("ratio", [0.0, 1e-8, 0.03, 0.5, 0.9, 0.999])
@pytest.mark.parametrize("mixed", [False, True])
def test_rho_one_dominant_eigenvalue(S, r, ratio, mixed):
    """The stop of the Lanczos process by dominance: lambda_1 = 1 (a positive eigenvector away
    from the all-ones start), one further eigenvalue `ratio`, the others ratio / 100 (mixed:
    spread between 0 and ratio), over and below where the stop is used."""
    rng = np.random.default_rng(r)
    v = 0.2 + rng.random(r)
    q, _ = np.linalg.qr(np.column_stack([v, rng.standard_normal((r, r - 1))]))
    lam = np.concatenate([[1.0, ratio], rng.random(r - 2) * ratio if mixed
                          else np.full(r - 2, ratio / 100)])
    G = 7.3e4 * (q * lam) @ q.T
    G = 0.5 * (G + G.T)
    got = S.rho(_t(G, torch.float64))
    ref = np.linalg.eigvalsh(G)[-1]
    assert abs(got - ref) <= 1e-13 * ref

@pytest.mark.parametrize("scale", [1e-140, 1e-100, 1e-84, 1e-60, 1e60, 1e100, 1e140])
def test_rho_dominance_at_any_scale(S, scale):
    """The stop by dominance does not depend on the scale of G: the products of squared
    off-diagonals it tests are formed relative to the gap."""
    rng = np.random.default_rng(20)
    P = rng.random((57, 20))
    G = P.T @ P
    got = S.rho(_t(G * scale, torch.float64)) / scale
    ref = np.linalg.eigvalsh(G)[-1]
    assert abs(got - ref) <= 1e-13 * ref


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,r,row", [(20999, 5, 3), (21000, 5, 3), (62999, 40, 3), (63000, 40, 3),
                                     (2100, 33, 4199)])
def test_rho_in_the_sparse_product(S, prec, n, r, row):
    """rho beside the sparse product, on both sides of the choice between the two forms of the
    launch (n < 15000 + 1200 r, fewer than 4e6 nonzeros), with no dominant eigenvalue (the
    partner's columns are nearly disjoint) and with one: FP64 1e-13; FP32 rounds P alone, the
    Gram of the rounded P is taken as the reference."""
    dt = torch.float64 if prec == "f64" else torch.float32
    rng = np.random.default_rng(n + r)
    k = (row - 1) // 2
    A = sp.diags([np.ones(n - d) for d in range(k + 1)], range(k + 1))
    A = (A + sp.triu(A, 1).T).tocsr()
    assert (A.nnz >= 4_000_000) == (row == 4199)
    for P in (rng.random((n, r)), 0.01 * rng.random((n, r))):
        if P.max() < 0.1:
            P[np.arange(n), np.arange(n) % r] += 1.0 + 0.1 * (np.arange(n) % r)
        Pt = _t(P, dt)
        with S.Plan(S.csr_from_scipy(A, dt), r, S.params(prec=S.prec_of(dt), max_outer=1)) as pl:
            got = pl.half_step(Pt.clone(), Pt, False)["rho"]
        Pd = Pt.double().cpu().numpy()
        ref = np.linalg.eigvalsh(Pd.T @ Pd)[-1]
        assert abs(got - ref) <= 1e-13 * ref


# ------------------------------------------------------------------ Gram and A-pass
# (132, 34) and (260, 64): FP32 workgroup chunks longer than a tile's K (one workgroup
# spans several tiles); (2048, 64), (4100, 34), (4608, 64): chunks that end inside tiles
@pytest.mark.parametrize("n,r", [(1, 1), (37, 5), (132, 34), (260, 64), (500, 10), (1029, 33),
                                 (2048, 64), (4100, 34), (4608, 64)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_gram_and_dense_apass(S, n, r, prec):
    rng = np.random.default_rng(n * 100 + r)
    A = rng.random((n, n))
    A = 0.5 * (A + A.T)
    P = rng.random((n, r))
    dt = torch.float64 if prec == "f64" else torch.float32
    At, Pt = _t(A, dt), _t(P, dt)
    A_in = At.double().cpu().numpy()       # identical (possibly rounded) inputs
    P_in = Pt.double().cpu().numpy()
    pl = S.Plan(S.dense(At), r, S.params(prec=S.F64 if prec == "f64" else S.F32, max_outer=1))
    G = pl.gram(Pt).cpu().numpy()
    assert nrel(G, P_in.T @ P_in) <= 1e-13
    B = torch.empty_like(Pt)
    pl.apass(Pt, B)
    tol = 1e-12 if prec == "f64" else 1e-5
    ref = O.apply_A(A_in, P_in)
    assert nrel(B.cpu().numpy(), ref) <= tol
    # A, P >= 0: every entry is a sum of nonnegative terms, |A||P| = A P
    assert comp_rel(B.cpu().numpy(), ref, ref) <= tol
    pl.close()


@pytest.mark.parametrize("n,r", [(64, 8), (500, 10), (1000, 32), (1100, 64), (2048, 40)])
def test_split_bf16_apass(S, n, r):
    rng = np.random.default_rng(7 + n)
    A = rng.random((n, n))
    A = 0.5 * (A + A.T)
    P = rng.random((n, r))
    At, Pt = _t(A, torch.float32), _t(P, torch.float32)
    A_in = At.double().cpu().numpy()
    P_in = Pt.double().cpu().numpy()
    pl = S.Plan(S.dense(At), r, S.params(prec=S.BF16X3, max_outer=1))
    B = torch.empty_like(Pt)
    pl.apass(Pt, B)
    ref = O.apply_A(A_in, P_in)
    err = nrel(B.cpu().numpy(), ref)
    # three-product split: operands exact to ~2^-16 relative, FP32 accumulation
    assert err <= 2e-5, err
    # entrywise: each operand's hi + lo is within 2^-17 of it, so every (nonnegative)
    # term is within ~2^-16 of its value, plus the FP32 sum: 3e-5 of A P per entry
    assert comp_rel(B.cpu().numpy(), ref, ref) <= 3e-5
    pl.close()


def _bf16_rne_bits(x32):
    u = x32.view(np.uint32).astype(np.uint64)
    r = (u + 0x7FFF + ((u >> 16) & 1)) >> 16
    return (r & 0xFFFF).astype(np.uint16)


def test_bf16_split_is_round_to_nearest_even(S):
    rng = np.random.default_rng(11)
    x = np.concatenate([rng.random(5000), rng.standard_normal(5000) * 1e3,
                        [0.0, -0.0, 1.0, 1.00390625, 1.005859375, 3.0e-39]]).astype(np.float32)
    hi, lo = S.split_bf16(_t(x, torch.float32))
    hi = hi.cpu().numpy().view(np.uint16)
    lo = lo.cpu().numpy().view(np.uint16)
    ref_hi = _bf16_rne_bits(x)
    hi_f = (ref_hi.astype(np.uint32) << 16).view(np.float32)
    ref_lo = _bf16_rne_bits((x - hi_f).astype(np.float32))
    assert np.array_equal(hi, ref_hi)
    assert np.array_equal(lo, ref_lo)
    recon = hi_f.astype(np.float64) + (ref_lo.astype(np.uint32) << 16).view(np.float32)
    rel = np.abs(recon - x) / np.maximum(np.abs(x), 1e-30)
    assert rel[np.abs(x) > 1e-30].max() <= 2.0 ** -16


# ------------------------------------------------------------------ CSR SpMM
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("r", [1, 7, 20, 32, 64])
def test_csr_spmm(S, prec, r):
    rng = np.random.default_rng(r)
    n = 3001
    a = sp.random(n, n, density=0.003, random_state=5, format="csr")
    a = (a + a.T + sp.diags(rng.random(n))).tolil()
    a[11, :] = rng.random(n) * (rng.random(n) < 0.5)  # one long row (~n/2 nonzeros)
    a[7, :] = 0                                       # an empty row
    a = a.tocsr()
    a.eliminate_zeros()
    a.sort_indices()
    assert a.indptr[8] == a.indptr[7]
    dt = torch.float64 if prec == "f64" else torch.float32
    M = S.csr_from_scipy(a, dt)
    X = _t(rng.random((n, r)), dt)
    Y = S.spmm(M, X)
    a_in = sp.csr_matrix((M.keep[2].double().cpu().numpy(), a.indices, a.indptr), shape=a.shape)
    ref = a_in @ X.double().cpu().numpy()
    tol = 1e-13 if prec == "f64" else 1e-6
    assert nrel(Y.cpu().numpy(), ref) <= tol
    mag = abs(a_in) @ np.abs(X.double().cpu().numpy())
    assert comp_rel(Y.cpu().numpy(), ref, mag) <= (1e-13 if prec == "f64" else 2e-6)


# ------------------------------------------------------------------ LAI product
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,ell,r", [(997, 16, 5), (20000, 74, 32), (5000, 128, 64),
                                    (70000, 16, 16)])
def test_lai_apass(S, prec, n, ell, r):
    rng = np.random.default_rng(n + ell)
    U, _ = np.linalg.qr(rng.standard_normal((n, ell)))
    lam = rng.standard_normal(ell) * 10
    P = rng.random((n, r))
    dt = torch.float64 if prec == "f64" else torch.float32
    Ut, Pt = _t(U, dt), _t(P, dt)
    lamt = _t(lam, torch.float64)
    pl = S.Plan(S.lowrank(Ut, lamt), r, S.params(prec=S.F64 if prec == "f64" else S.F32,
                                                  max_outer=1, validate=0))
    B = torch.empty_like(Pt)
    pl.apass(Pt, B)
    ref = O.apply_A(O.LowRank(Ut.double().cpu().numpy(), lam), Pt.double().cpu().numpy())
    tol = 1e-12 if prec == "f64" else 2e-6
    assert nrel(B.cpu().numpy(), ref) <= tol
    # entrywise against |U| |lam| |U|^T |P| (U has mixed signs: the products cancel)
    Ua = np.abs(Ut.double().cpu().numpy())
    mag = Ua @ (np.abs(lam)[:, None] * (Ua.T @ np.abs(Pt.double().cpu().numpy())))
    assert comp_rel(B.cpu().numpy(), ref, mag) <= (1e-13 if prec == "f64" else 2e-6)
    pl.close()


@pytest.mark.parametrize("n,r,pad", [(16, 16, 0), (17, 17, 1), (127, 3, 0), (128, 32, 3),
                                     (129, 33, 0), (257, 48, 1), (1000, 49, 0), (2500, 20, 7),
                                     (4095, 5, 0), (4097, 64, 1), (4100, 17, 0)])
def test_dense_apass_f64_edges(S, n, r, pad):
    """The FP64 product at the edges of its tiles (16 and 32 rows, 16 columns), its K splits
    and the wavefronts' quarters; padding columns (odd leading dimensions among them) hold
    NaN and must not be read into the result.  The product adds n terms in FP64:
    |error| <= n 2^-53 sum |a| |p| entrywise (both sides), 1e-12 normwise."""
    rng = np.random.default_rng(n + r)
    A = rng.random((n, n))
    A = 0.5 * (A + A.T)
    buf = torch.full((n, n + pad), float("nan"), dtype=torch.float64, device=DEV)
    buf[:, :n] = torch.from_numpy(A).to(DEV)
    P = rng.random((n, r))
    Pt = torch.from_numpy(P).to(DEV)
    with S.Plan(S.dense(buf[:, :n]), r, S.params(prec=S.F64, max_outer=1)) as pl:
        B = torch.empty_like(Pt)
        pl.apass(Pt, B)
    assert nrel(B.cpu().numpy(), A @ P) <= 1e-12


@pytest.mark.parametrize("n,r,pad", [(15, 1, 0), (16, 15, 1), (33, 32, 0), (65, 5, 0), (255, 31, 1),
                                     (257, 33, 0), (1000, 20, 0), (1001, 35, 2), (3001, 21, 0),
                                     (5000, 32, 1), (8190, 63, 0)])
def test_dense_apass_f32_edges(S, n, r, pad):
    """The general FP32 product (r <= 32, or odd r or n): K ranges of fewer, as many and more
    batches than are in flight, remainders of single rows, edges of the 32-column blocks;
    padding columns hold NaN and must not be read into the result.  Sums of n nonnegative
    terms in FP32: |error| <= n 2^-24 of the entry."""
    rng = np.random.default_rng(n + r)
    A = rng.random((n, n), dtype=np.float32)
    A = np.triu(A) + np.triu(A, 1).T
    buf = torch.full((n, n + pad), float("nan"), dtype=torch.float32, device=DEV)
    buf[:, :n] = torch.from_numpy(A).to(DEV)
    P = rng.random((n, r), dtype=np.float32)
    Pt = torch.from_numpy(P).to(DEV)
    with S.Plan(S.dense(buf[:, :n]), r, S.params(prec=S.F32, max_outer=1)) as pl:
        B = torch.empty_like(Pt)
        pl.apass(Pt, B)
    ref = A.astype(np.float64) @ P.astype(np.float64)
    assert (np.abs(B.cpu().numpy() - ref) <= n * 2.0 ** -24 * ref).all()


@pytest.mark.parametrize("n,r", [(33, 16), (200, 16), (1000, 40), (4100, 17)])
def test_dense_apass_f64_infinite_partner(S, n, r):
    """An infinite entry of P makes its column of A P infinite (A > 0), never NaN, wherever it
    lies in the K ranges: the zeros that fill a range's end meet zeros, not a row of P."""
    rng = np.random.default_rng(n)
    A = rng.random((n, n)) + 0.1
    A = 0.5 * (A + A.T)
    P = rng.random((n, r))
    rows = np.unique(np.linspace(0, n - 1, r - 1).astype(int))
    P[rows, np.arange(len(rows))] = np.inf     # the last row among them
    Pt = _t(P, torch.float64)
    with S.Plan(S.dense(_t(A, torch.float64)), r, S.params(prec=S.F64, max_outer=1)) as pl:
        B = torch.empty_like(Pt)
        pl.apass(Pt, B)
    B = B.cpu().numpy()
    assert (B[:, : len(rows)] == np.inf).all()
    assert nrel(B[:, len(rows):], A @ P[:, len(rows):]) <= 1e-12
