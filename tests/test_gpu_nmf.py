"""GPU parity of NMPBB for rectangular NMF (snmf_nmf_solve, eq. (1.1) with the
alternating scheme of Section 2.1) against the oracle (oracle/nmf.py) from the same V, W0
and Ht0.

Dense FP32 products run on the matrix cores as split-K panels (several K chunks with
ragged last chunks in every dense case here; r = 40 and 64 take two MFMA column blocks).

Tolerances: FP64 runs the oracle's arithmetic in another summation order, so ten outer
iterations agree to 1e-8 relative (factors and residual trace; measured 1e-13 at r <= 12
and 1e-9 at r = 64, where the BB steps carry the 1e-15 differences of longer sums
further).  FP32 sums in FP32 with FP64 scalars: the factors agree to 2e-3 normwise and the residual trace to 5e-4 relative
to its largest value.  Their FP32 sources are the products (split-K panels on the matrix
cores, about 1e-6 relative per entry, added in FP32) and the gradient carried by
linearity, which the BB steps amplify: the FP32 rounding model (every array rounded to
FP32 on the oracle's iteration) moves the 3-iteration result at r = 64 by 5e-5, the GPU's
measured 1.8e-4 (factors) and 1.3e-4 (trace); at r <= 33 over 10 iterations at most 5.5e-5
and 4.4e-5.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle as O
from paper_2606_02887_amd import gen
from parity_util import nrel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"
DT = {"f64": torch.float64, "f32": torch.float32}
TOL = {"f64": (1e-8, 1e-8), "f32": (2e-3, 5e-4)}   # (factors, residual trace)


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_02887_amd import snmf
    return snmf


def _run(S, kind, prec, m, n, r, seed, outer):
    dt = DT[prec]
    if kind == "dense":
        prob = gen.planted_rect(m, n, r, seed)
        Vt = torch.from_numpy(prob["V"]).to(DEV, dt)
        M = S.dense(Vt)
        Vref = Vt.double().cpu().numpy()
    else:
        prob = gen.random_rect_csr(m, n, 0.02, r, seed)
        M = S.csr_from_scipy(prob["V"], dt)
        Vref = prob["V"].copy().astype(np.float64)
        Vref.data = M.keep[2].double().cpu().numpy()
    W0 = torch.from_numpy(prob["W0"]).to(DEV, dt)
    H0 = torch.from_numpy(prob["Ht0"]).to(DEV, dt)
    W, Ht, info = S.nmf_solve(M, n, W0, H0, S.params(prec=S.prec_of(dt), lam=0.0, max_outer=outer))
    W0n, H0n = W0.double().cpu().numpy(), H0.double().cpu().numpy()
    Wo, Ho, hist = O.nmf_solve(Vref, W0n, H0n, O.Params(), outer)
    return W, Ht, info, Wo, Ho, hist, (Vref, W0n, H0n)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind,m,n,r", [("dense", 700, 450, 12), ("dense", 130, 1029, 5),
                                        ("dense", 3000, 1500, 64), ("dense", 2049, 777, 40),
                                        ("csr", 3000, 1700, 16), ("csr", 517, 2048, 33)])
def test_nmf_matches_oracle(S, prec, kind, m, n, r):
    # FP32 at r = 40 and 64: 3 outer iterations (the FP32 arithmetic alone, modelled on
    # the oracle with every array rounded to FP32, moves the 10-iteration result by 1.1e-3
    # at r = 64 and 1.8e-2 at r = 40: the iteration amplifies rounding-size differences
    # there; FP64 checks the same cases over 10 iterations)
    outer = 3 if (prec == "f32" and r > 32) else 10
    W, Ht, info, Wo, Ho, hist, inputs = _run(S, kind, prec, m, n, r, 11 + m, outer)
    ftol, rtol = TOL[prec]
    res_o = np.array([h["res_WH"] for h in hist])
    Wg, Hg = W.double().cpu().numpy(), Ht.double().cpu().numpy()
    ew, eh = nrel(Wg, Wo), nrel(Hg, Ho)
    tr = info["trace"]
    pg_o = np.array([h["pg"] for h in hist])
    eres = np.abs(tr[:, 0] - res_o).max() / res_o.max()
    epg = abs(info["pg_norm"] - pg_o[-1]) / pg_o[-1]
    print(f"{kind} {m}x{n} r={r} {prec}: W {ew:.1e}, Ht {eh:.1e}, residual trace {eres:.1e}, "
          f"pg {epg:.1e}; residual {res_o[0]:.4f} -> {res_o[-1]:.4f}")
    assert info["status"] == 0 and info["outer"] == outer and tr.shape[0] == outer
    assert ew <= ftol and eh <= ftol
    assert eres <= rtol
    # the objective is res^2 ||V||^2 / 2 on both sides: its relative error is twice the
    # residual's at the last record, where the trace tolerance (relative to the largest
    # residual) is res_max / res_last times larger
    obj_o = hist[-1]["objective"]
    assert abs(info["objective"] - obj_o) <= 2.5 * rtol * res_o.max() / res_o[-1] * obj_o
    assert epg <= (1e-7 if prec == "f64" else 0.05)
    assert np.isnan(info["res_WWt"]) and np.isnan(tr[:, 1]).all()
    assert (Wg >= 0).all() and (Hg >= 0).all()


def test_nmf_reaches_planted_fit(S):
    """200 outer iterations on the planted dense problem (m = 700, n = 450, r = 12, noise
    1%) in FP32 bring the residual to the noise level, as the oracle's 200 iterations do
    (both below 0.02, within 5% of each other)."""
    W, Ht, info, Wo, Ho, hist, _ = _run(S, "dense", "f32", 700, 450, 12, 711, 200)
    print(f"200 outer: gpu {info['res_WH']:.5f}, oracle {hist[-1]['res_WH']:.5f}")
    assert info["res_WH"] < 0.02 and hist[-1]["res_WH"] < 0.02
    assert abs(info["res_WH"] - hist[-1]["res_WH"]) <= 0.05 * hist[-1]["res_WH"]


def test_nmf_error_codes(S):
    V = torch.rand((40, 30), dtype=torch.float64, device=DEV)
    W0 = torch.rand((40, 4), dtype=torch.float64, device=DEV)
    H0 = torch.rand((30, 4), dtype=torch.float64, device=DEV)

    def code(M, ncols, W, H, **kw):
        kw.setdefault("prec", S.prec_of(torch.float64))
        with pytest.raises(S.SnmfError) as e:
            S.nmf_solve(M, ncols, W, H, S.params(max_outer=3, **kw))
        return e.value.name

    assert code(S.dense(V), 30, W0, H0, lam=0.5) == "E_ARG"
    assert code(S.dense(V), 31, W0, torch.rand((31, 4), dtype=torch.float64, device=DEV),
                lam=0.0) == "E_SHAPE"                                  # ld 30 < n_cols
    assert code(S.dense(V), 30, W0, H0, lam=0.0, prec=S.BF16X3) == "E_UNSUPPORTED"
    Vn = V.clone()
    Vn[3, 4] = -1.0
    assert code(S.dense(Vn), 30, W0, H0, lam=0.0) == "E_NEGATIVE"
    a = sp.random(40, 30, density=0.2, random_state=3, format="csr")
    M = S.csr_from_scipy(a, torch.float64)
    assert code(M, 20, W0, H0[:20].contiguous(), lam=0.0) == "E_SHAPE"   # columns >= n_cols
    lr = S.lowrank(W0, torch.ones(4, dtype=torch.float64, device=DEV))
    assert code(lr, 30, W0, H0, lam=0.0) == "E_UNSUPPORTED"


@pytest.mark.parametrize("m,n,r", [(64, 64, 64), (100, 516, 34), (129, 260, 36), (513, 132, 62),
                                   (700, 1028, 64), (1300, 508, 48), (2048, 2052, 34),
                                   (515, 640, 40), (4099, 1600, 64)])
@pytest.mark.parametrize("pad", [0, 8])
def test_nmf_wide_products_same_bits(S, m, n, r, pad):
    """r in (32, 64], even, on aligned V: both products read V through the wide kernels, each
    sum over the same panels in the same order as the general path, which a leading
    dimension not divisible by 4 selects: the factors are bitwise equal.  Edges: rows not
    divisible by the 128 of a wavefront, last panels of fewer than 16 k, pitched V (its
    padding NaN)."""
    prob = gen.planted_rect(m, n, r, 3 * m + n)
    out = []
    for ld in (n + pad, n + pad + 1):
        buf = torch.full((m, ld), float("nan"), dtype=torch.float32, device=DEV)
        buf[:, :n] = torch.from_numpy(prob["V"]).to(DEV)
        W, Ht, info = S.nmf_solve(S.dense(buf[:, :n]), n,
                                  torch.from_numpy(prob["W0"]).to(DEV, torch.float32),
                                  torch.from_numpy(prob["Ht0"]).to(DEV, torch.float32),
                                  S.params(prec=S.F32, lam=0.0, max_outer=2))
        assert info["status"] == 0
        out.append((W, Ht))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
