"""Step-level (lockstep) and whole-solve parity of the HIP SNMPBB path against the oracle.

Lockstep: both sides start a half-step from the same (X, P) and run the same number of
inner iterations; the results must agree to 1e-12 (FP64) / 1e-5 (FP32) normwise, and
the device scalars (rho, final BB step, accepted beta, <S,S>, <S,Y>) must match.
Whole solve: final residual ||A - W H||/||A|| and projected-gradient norm within 1e-3
relative of the oracle (1e-9 in FP64) after the same number of outer iterations, at a
budget before the iteration amplifies rounding differences; at longer budgets the end
point must lie inside the envelope of oracle runs from rounding-level perturbed starts.
"""
import json
import os
import time

import numpy as np
import pytest
import scipy.sparse as sp

import oracle as O
from paper_2606_02887_amd import gen
from parity_util import elem_rel, nrel, rel
from rounding_model import half_step_fp32

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def S():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_02887_amd import snmf
    return snmf


def _t(x, dtype):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV, dtype)


DT = {"f64": torch.float64, "f32": torch.float32}


# entrywise bound beside the normwise one: |a - b| <= ETOL (|b| + 1e-3 max|b|)
ETOL = {"f64": 1e-10, "f32": 1e-4}


def fp32_bounds(Aop, X, P, prm, L=None, laplacian=False):
    """Normwise and entrywise FP32 bounds of a half-step: 1e-5 and 1e-4, or 3x and 10x
    what FP32 rounding of the gradient-by-linearity update alone moves X+ from the oracle
    (tests/rounding_model.py), whichever is larger.  That movement is far below 1e-5 for
    most inputs; where the partner's columns are strongly correlated it grows with n
    (about 1.6e-5 at n = 70000, r = 16)."""
    import oracle as O_
    hs = O_.HalfStep(Aop, P, prm.lam, prm.gamma if laplacian else 0.0, L if laplacian else None)
    Xo = O_.nmpbb(hs, X, prm)
    Xm = half_step_fp32(O_.HalfStep(Aop, P, prm.lam, prm.gamma if laplacian else 0.0,
                                    L if laplacian else None), X, prm)
    return max(1e-5, 3.0 * nrel(Xm, Xo)), max(ETOL["f32"], 10.0 * elem_rel(Xm, Xo))


def _prec(S, p):
    return {"f64": S.F64, "f32": S.F32, "bf16x3": S.BF16X3}[p]


def _lockstep(S, Aop_gpu, Aop_oracle, X, P, prec, is_hstep, lam, gamma=0.0, L_gpu=None,
              L_or=None, inner=5):
    dt = DT["f32" if prec == "bf16x3" else prec]
    Xt, Pt = _t(X, dt), _t(P, dt)
    X_in, P_in = Xt.double().cpu().numpy(), Pt.double().cpu().numpy()
    prm = S.params(lam=lam, gamma=gamma, prec=_prec(S, prec), inner_iters=inner, max_outer=1,
                   validate=0)
    pl = S.Plan(Aop_gpu, X.shape[1], prm, L_gpu)
    sc = pl.half_step(Xt, Pt, bool(is_hstep))
    pl.close()
    log = []
    oprm = O.Params(lam=lam, gamma=gamma, inner_iters=inner)
    lap = bool(is_hstep) and L_or is not None
    Xo = O.half_step(Aop_oracle, X_in, P_in, oprm, laplacian=lap, L=L_or, log=log)
    if prec == "f64":
        bounds = (1e-12, ETOL["f64"])
    else:
        bounds = fp32_bounds(Aop_oracle, X_in, P_in, oprm, L_or, lap)
    Xg = Xt.double().cpu().numpy()
    print(f"lockstep {prec} n={X.shape[0]} r={X.shape[1]} h={is_hstep}: nrel {nrel(Xg, Xo):.3e} "
          f"entrywise {elem_rel(Xg, Xo):.3e} (bounds {bounds[0]:.2e}, {bounds[1]:.2e})")
    _lockstep.bounds = bounds
    return Xg, Xo, sc, log


def _check_scalars(sc, log, tol):
    last = log[-1]
    assert abs(sc["rho"] - log[0]["rho"]) <= tol * log[0]["rho"]
    assert abs(sc["alpha"] - last["alpha"]) <= tol * last["alpha"]
    assert abs(sc["beta"] - last["beta"]) <= tol
    assert abs(sc["ss"] - last["ss"]) <= tol * max(last["ss"], 1e-300) + 1e-300
    assert abs(sc["sy"] - last["sy"]) <= tol * max(abs(last["sy"]), 1e-300) + 1e-300
    assert int(sc["ls_evals"]) == sum(e["evals"] for e in log)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("is_hstep", [0, 1])
@pytest.mark.parametrize("n,r", [(300, 8), (700, 33)])
def test_half_step_lockstep_dense(S, prec, is_hstep, n, r):
    prob = gen.planted_dense(n, r, 101 + n)
    A = prob["A"]
    rng = np.random.default_rng(5)
    X = prob["W0"]
    P = np.maximum(prob["Wstar"] + 0.05 * rng.standard_normal((n, r)), 0)
    At = _t(A, DT[prec])
    A_in = At.double().cpu().numpy()
    lam = O.default_lambda(A_in)
    Xg, Xo, sc, log = _lockstep(S, S.dense(At), A_in, X, P, prec, is_hstep, lam)
    tol, etol = _lockstep.bounds
    assert nrel(Xg, Xo) <= tol
    assert elem_rel(Xg, Xo) <= etol
    _check_scalars(sc, log, 1e-10 if prec == "f64" else 1e-4)
    assert (Xg >= 0).all()


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_half_step_lockstep_graph_laplacian(S, prec):
    """H-step of Graph-SNMPBB: gradient term gam L Ht and the <D, L D> curvature."""
    p = gen.sbm_problem(n=600, k=4, r=4, p_in=0.1, p_out=0.01, seed=17)
    A, L = p["A"], O.knn_laplacian(p["X"], p["knn"])
    rng = np.random.default_rng(2)
    X = p["W0"]
    P = rng.random(X.shape) * X.mean()
    dt = DT[prec]
    Ag, Lg = S.csr_from_scipy(A, dt), S.csr_from_scipy(L, dt)
    A_in = sp.csr_matrix((Ag.keep[2].double().cpu().numpy(), A.indices, A.indptr), A.shape)
    L_in = sp.csr_matrix((Lg.keep[2].double().cpu().numpy(), L.indices, L.indptr), L.shape)
    lam = O.default_lambda(A_in)
    Xg, Xo, sc, log = _lockstep(S, Ag, A_in, X, P, prec, 1, lam, gamma=0.2, L_gpu=Lg, L_or=L_in)
    tol, etol = _lockstep.bounds
    assert nrel(Xg, Xo) <= tol
    assert elem_rel(Xg, Xo) <= etol
    _check_scalars(sc, log, 1e-10 if prec == "f64" else 1e-4)


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_half_step_lockstep_lai(S, prec):
    n, ell, r = 3000, 24, 6
    a = gen.powerlaw_csr(n=n, seed=9)
    U, lam_ = O.range_finder(a, ell, 2, gen.sketch_matrix(n, ell + 6, 3))
    rng = np.random.default_rng(4)
    X = rng.random((n, r)) * 0.05
    P = rng.random((n, r)) * 0.05
    dt = DT[prec]
    Ut = _t(U, dt)
    lr_in = O.LowRank(Ut.double().cpu().numpy(), lam_)
    lam = O.default_lambda(lr_in)
    Xg, Xo, sc, log = _lockstep(S, S.lowrank(Ut, _t(lam_, torch.float64)), lr_in, X, P, prec, 0,
                                lam)
    tol, etol = _lockstep.bounds
    assert nrel(Xg, Xo) <= tol
    assert elem_rel(Xg, Xo) <= etol
    _check_scalars(sc, log, 1e-10 if prec == "f64" else 1e-4)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("is_hstep", [0, 1])
def test_half_step_lockstep_lai_large_arrays(S, prec, is_hstep):
    """n x r arrays of at least 4 MiB (n = 70000, r = 16): step 1 keeps D in registers
    only and step 2 forms it again; several row tiles per workgroup.  FP64 is held to
    1e-12.  In FP32 the A-pass itself is exact to 1.1e-7 (test_lai_apass_large), but the
    partner here (0.05 U[0,1], columns strongly correlated) makes the first projection
    cancel most of X, so the FP32 rounding of the gradient update is large against
    grad f(Z) and grows with n; the rounding model moves X+ by 1.6e-5 (measured on the GPU:
    2.2e-5, spread evenly over the row tiles, and 1.4 to 2.5 times the model at every n
    from 3000 to 70000), hence the bound of fp32_bounds."""
    n, ell, r = 70000, 16, 16
    a = gen.powerlaw_csr(n=n, seed=9)
    U, lam_ = O.range_finder(a, ell, 2, gen.sketch_matrix(n, ell + 6, 3))
    rng = np.random.default_rng(6)
    X = rng.random((n, r)) * 0.05
    P = rng.random((n, r)) * 0.05
    dt = DT[prec]
    Ut = _t(U, dt)
    lr_in = O.LowRank(Ut.double().cpu().numpy(), lam_)
    lam = O.default_lambda(lr_in)
    Xg, Xo, sc, log = _lockstep(S, S.lowrank(Ut, _t(lam_, torch.float64)), lr_in, X, P, prec,
                                is_hstep, lam)
    tol, etol = _lockstep.bounds
    assert nrel(Xg, Xo) <= tol
    assert elem_rel(Xg, Xo) <= etol
    _check_scalars(sc, log, 1e-10 if prec == "f64" else 1e-4)


def test_half_step_ragged_rank_and_tail(S):
    """r = 1 and n not a multiple of any tile: exact FP64 agreement."""
    prob = gen.planted_dense(517, 1, 3)
    A = prob["A"]
    rng = np.random.default_rng(1)
    P = rng.random((517, 1))
    Xg, Xo, sc, log = _lockstep(S, S.dense(_t(A, torch.float64)), A, prob["W0"], P, "f64", 0,
                                O.default_lambda(A), inner=9)
    assert nrel(Xg, Xo) <= 1e-12


# ------------------------------------------------------------------ whole solves
def _whole(S, A_gpu, A_or, W0, prec, outer, lam, gamma=0.0, L_gpu=None, L_or=None):
    dt = DT["f32" if prec == "bf16x3" else prec]
    W0t = _t(W0, dt)
    prm = S.params(lam=lam, gamma=gamma, prec=_prec(S, prec), max_outer=outer)
    W, Ht, info = S.solve(A_gpu, W0t, prm, L_gpu)
    _, _, hist = O.snmpbb(A_or, W0t.double().cpu().numpy(), O.Params(lam=lam, gamma=gamma), outer,
                          L=L_or)
    return W.double().cpu().numpy(), Ht.double().cpu().numpy(), info, hist


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
def test_whole_solve_config0_point(S, prec):
    """Config 0 (planted dense n=500, r=10) for 20 outer iterations: a budget at which
    rounding-level differences have not yet been amplified by the iteration (the
    oracle's own spread under 1e-7 relative perturbations of W0 is below 1e-7 there and
    grows to ~1e-3 by 40 iterations)."""
    prob = gen.config(0)
    A = prob["A"]
    dt = DT["f32" if prec == "bf16x3" else prec]
    At = _t(A, dt)
    A_in = At.double().cpu().numpy()
    lam = O.default_lambda(A_in)
    W, Ht, info, hist = _whole(S, S.dense(At), A_in, prob["W0"], prec, 20, lam)
    ref = hist[-1]
    assert info["outer"] == 20 and info["status"] == 0
    tol = 1e-9 if prec == "f64" else 1e-3
    assert abs(info["res_WH"] - ref["res_WH"]) <= tol * ref["res_WH"]
    assert abs(info["pg_norm"] - ref["pg"]) <= tol * ref["pg"]
    assert rel(info["res_WWt"], ref["res_WWt"]) <= tol
    assert rel(info["objective"], ref["objective"]) <= tol
    assert rel(info["sym_gap"], ref["sym_gap"]) <= tol
    # the device monitor vs the FP64 residual of the returned factors: FP64 to rounding;
    # FP32 to ~1e-4 (FP32 A-pass in the cross term <A W, Ht>); split BF16 measures against
    # A_hi + A_lo, whose 2^-17 elementwise error shifts the cross term by ~1e-4 of res^2
    direct = O.residual_WH(A_in, W, Ht)
    mtol = {"f64": 1e-10, "f32": 1e-4, "bf16x3": 5e-4}[prec]
    assert abs(info["res_WH"] - direct) <= mtol * direct
    assert (W >= 0).all() and (Ht >= 0).all()
    assert np.all(np.diff(info["trace"][:, 5]) >= 0)


@pytest.fixture(scope="module")
def config0_ensemble():
    """The oracle's config-0 runs for 500 outer iterations from W0 and from 31
    rounding-level (2^-24 relative) changes of it (tests/golden/c0_ensemble.json, written
    by make_c0_ensemble.py from the oracle alone): their spread measures how far the
    iteration itself carries rounding differences by that budget."""
    with open(os.path.join(GOLDEN, "c0_ensemble.json")) as f:
        ens = json.load(f)
    prob = gen.config(0)
    assert ens["outer"] == 500 and abs(ens["lambda"] - O.default_lambda(prob["A"])) <= 1e-12 * ens["lambda"]
    runs = ens["runs"]
    return prob, ens["lambda"], {k: np.array([r_[k] for r_ in runs])
                                 for k in ("res_WH", "res_WWt", "pg", "objective")}


def _ensemble_starts(W0, count, seed0=100):
    """count starts W0 * (1 + 2^-22 u), u = +-1 (a change an FP32 copy keeps), seeded."""
    return np.stack([W0 * (1.0 + 2.0 ** -22 * np.random.default_rng(seed0 + s).choice(
        [-1.0, 1.0], size=W0.shape)) for s in range(count)])


def _z(gpu, ora):
    """Two-sample z statistic of the difference of the means."""
    se = np.sqrt(np.var(gpu, ddof=1) / gpu.size + np.var(ora, ddof=1) / ora.size)
    return abs(gpu.mean() - ora.mean()) / max(se, 1e-300)


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
def test_whole_solve_config0_ensemble(S, prec, config0_ensemble):
    """500 outer iterations, where the iteration has spread rounding-level differences of
    the start over its attractor (the oracle's 32 runs: residuals and objective within
    0.3%, the projected-gradient norm from 2.3 to 6.9).  The GPU form runs 16 rounding-
    level changes of the start in one batch; each end-point measure (residuals, objective,
    log of the projected-gradient norm) must have a mean within 4 standard errors of the
    oracle ensemble's.  The split-BF16 form multiplies A_hi + A_lo, a 2^-17 change of A,
    so it is also held to 3e-3 of the oracle mean in the residuals and objective."""
    prob, lam, ens = config0_ensemble
    dt = DT["f32" if prec == "bf16x3" else prec]
    A = _t(prob["A"], dt)
    W0s = _t(_ensemble_starts(prob["W0"], 16), dt)
    with S.Batch([S.dense(A)], [prob["W0"].shape[1]],
                 S.params(lam=lam, prec=_prec(S, prec), max_outer=500), 16, lam=[lam]) as b:
        _, _, infos, _ = b.solve([W0s])
    assert all(i["outer"] == 500 and i["status"] == 0 for i in infos)
    gpu = {k: np.array([i[{"pg": "pg_norm"}.get(k, k)] for i in infos]) for k in ens}
    for k in ens:
        g, o = (np.log(gpu[k]), np.log(ens[k])) if k == "pg" else (gpu[k], ens[k])
        z = _z(g, o)
        print(f"{prec} {k}: gpu mean {gpu[k].mean():.6g} sd {gpu[k].std():.3g}; oracle mean "
              f"{ens[k].mean():.6g} sd {ens[k].std():.3g}; z {z:.2f}")
        assert z <= 4.0, (k, z)
        if k != "pg" and prec == "bf16x3":
            assert rel(gpu[k].mean(), ens[k].mean()) <= 3e-3


def test_whole_solve_trace_matches_oracle_history(S):
    prob = gen.planted_dense(200, 5, 44)
    A = prob["A"]
    lam = O.default_lambda(A)
    W, Ht, info, hist = _whole(S, S.dense(_t(A, torch.float64)), A, prob["W0"], "f64", 40, lam)
    tr = info["trace"]
    ores = np.array([h["res_WH"] for h in hist])
    opg = np.array([h["pg"] for h in hist])
    osym = np.array([h["sym_gap"] for h in hist])
    orww = np.array([h["res_WWt"] for h in hist])
    oobj = np.array([h["objective"] for h in hist])
    assert np.abs(tr[:, 0] - ores).max() <= 1e-9 * ores.max()
    assert np.abs(tr[:, 1] - orww).max() <= 1e-9 * orww.max()
    assert np.abs(tr[:, 3] - opg).max() <= 1e-6 * opg.max()
    assert np.abs(tr[:, 2] - osym).max() <= 1e-9
    assert np.abs(tr[:, 4] - oobj).max() <= 1e-9 * oobj.max()


def test_whole_solve_graph(S):
    p = gen.sbm_problem(n=1000, k=5, r=5, p_in=0.08, p_out=0.004, seed=23)
    A, L = p["A"], O.knn_laplacian(p["X"], p["knn"])
    Ag, Lg = S.csr_from_scipy(A, torch.float64), S.csr_from_scipy(L, torch.float64)
    lam = O.default_lambda(A)
    W, Ht, info, hist = _whole(S, Ag, A, p["W0"], "f64", 60, lam, gamma=0.2, L_gpu=Lg, L_or=L)
    ref = hist[-1]
    assert abs(info["res_WH"] - ref["res_WH"]) <= 1e-3 * ref["res_WH"]
    assert abs(info["pg_norm"] - ref["pg"]) <= 1e-3 * ref["pg"]


def test_whole_solve_lai(S):
    n = 5000
    a = gen.powerlaw_csr(n=n, seed=31)
    U, lam_ = O.range_finder(a, 32, 2, gen.sketch_matrix(n, 42, 5))
    lr = O.LowRank(U, lam_)
    rng = np.random.default_rng(8)
    W0 = gen.start_factor(rng, n, 8, gen.mean_of_sparse(a))
    lam = O.default_lambda(lr)
    W, Ht, info, hist = _whole(S, S.lowrank(_t(U, torch.float64), _t(lam_, torch.float64)), lr,
                               W0, "f64", 30, lam)
    ref = hist[-1]
    assert abs(info["res_WH"] - ref["res_WH"]) <= 1e-3 * ref["res_WH"]


def test_target_residual_stops_early(S):
    prob = gen.planted_dense(300, 6, 9)
    A = prob["A"]
    lam = O.default_lambda(A)
    _, _, hist = O.snmpbb(A, prob["W0"], O.Params(lam=lam), 200)
    tgt = hist[30]["res_WH"]
    prm = S.params(lam=lam, prec=S.F64, max_outer=200, target_res=tgt, check_every=4)
    W, Ht, info = S.solve(S.dense(_t(A, torch.float64)), _t(prob["W0"], torch.float64), prm)
    first = next(i for i, h in enumerate(hist) if h["res_WH"] <= tgt) + 1
    assert info["converged_at"] == first == info["outer"]
    assert info["seconds_to_target"] > 0


def test_deterministic_bitwise(S):
    prob = gen.planted_dense(400, 12, 10)
    At = _t(prob["A"], torch.float32)
    W0 = _t(prob["W0"], torch.float32)
    prm = S.params(lam=O.default_lambda(prob["A"]), max_outer=30)
    W1, H1, _ = S.solve(S.dense(At), W0, prm)
    W2, H2, _ = S.solve(S.dense(At), W0, prm)
    assert torch.equal(W1, W2) and torch.equal(H1, H2)


def test_graph_replay_equals_direct_launches(S):
    prob = gen.planted_dense(300, 7, 12)
    At = _t(prob["A"], torch.float32)
    W0 = _t(prob["W0"], torch.float32)
    lam = O.default_lambda(prob["A"])
    Wa, Ha, ia = S.solve(S.dense(At), W0, S.params(lam=lam, max_outer=25, use_graph=1))
    Wb, Hb, ib = S.solve(S.dense(At), W0, S.params(lam=lam, max_outer=25, use_graph=0))
    assert torch.equal(Wa, Wb) and torch.equal(Ha, Hb)
    assert np.array_equal(ia["trace"][:, :5], ib["trace"][:, :5])


# ------------------------------------------------------------------ error paths
def test_error_codes(S):
    prob = gen.planted_dense(50, 3, 1)
    A = prob["A"].copy()
    W0 = prob["W0"].copy()
    prm = S.params(prec=S.F64, max_outer=2)
    bad = W0.copy()
    bad[3, 1] = np.nan
    with pytest.raises(S.SnmfError) as e:
        S.solve(S.dense(_t(A, torch.float64)), _t(bad, torch.float64), prm)
    assert e.value.name == "E_NONFINITE"
    neg = A.copy()
    neg[2, 5] = neg[5, 2] = -1.0
    with pytest.raises(S.SnmfError) as e:
        S.solve(S.dense(_t(neg, torch.float64)), _t(W0, torch.float64), prm)
    assert e.value.name == "E_NEGATIVE"
    a = sp.random(60, 60, density=0.1, random_state=1, format="csr")
    with pytest.raises(S.SnmfError) as e:
        S.solve(S.csr_from_scipy(a, torch.float64), _t(np.ones((60, 3)), torch.float64), prm)
    assert e.value.name == "E_NOT_SYMMETRIC"
    z = np.zeros((50, 3))
    with pytest.raises(S.SnmfError) as e:
        S.solve(S.dense(_t(A, torch.float64)), _t(z, torch.float64), prm)
    assert e.value.name == "E_BREAKDOWN"


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_dense_symmetry_check_is_opt_in(S, prec):
    """params.check_symmetry: a dense A with one mirrored pair apart (by 1e-3 relative)
    gives E_NOT_SYMMETRIC with the check and solves without it; a product X X^T formed on
    the device (mirrored entries equal up to its rounding) passes the check, in a plan and
    in a batch."""
    dt = DT[prec]
    p = S.F64 if prec == "f64" else S.F32
    prob = gen.planted_dense(90, 3, 21)
    A = prob["A"].copy()
    A[3, 70] *= 1.001
    W0 = _t(prob["W0"], dt)
    with pytest.raises(S.SnmfError) as e:
        S.solve(S.dense(_t(A, dt)), W0, S.params(prec=p, max_outer=2, check_symmetry=1))
    assert e.value.name == "E_NOT_SYMMETRIC"
    with pytest.raises(S.SnmfError) as e:
        S.Batch([S.dense(_t(A, dt))], [3], S.params(prec=p, max_outer=2, check_symmetry=1), 1)
    assert e.value.name == "E_NOT_SYMMETRIC"
    _, _, info = S.solve(S.dense(_t(A, dt)), W0, S.params(prec=p, max_outer=2))
    assert info["status"] == 0
    X = torch.rand((300, 7), dtype=dt, device=DEV)
    Ag = (X @ X.T).contiguous()
    _, _, info = S.solve(S.dense(Ag), X.contiguous(), S.params(prec=p, max_outer=1,
                                                             check_symmetry=1))
    assert info["status"] == 0


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_exact_stationary_start_stops_and_keeps_the_monitor(S, prec):
    """Integer planted factors with lambda = 0 make every product exact, so W* is an exact
    stationary point: the first inner iteration of each half-step gives S = 0 and the
    later iterations stop (Algorithm 1 reaches <S,S> = 0).  The monitor record of the
    stopped H-step must still be the final iterate's: zero residual and PG norm, and the
    factors unchanged."""
    rng = np.random.default_rng(5)
    n, r = 70, 3
    Wt = rng.integers(0, 3, size=(n, r)).astype(np.float64)
    Wt[np.arange(r), np.arange(r)] = 2.0           # full column rank
    A = Wt @ Wt.T
    dt = torch.float32 if prec == "f32" else torch.float64
    p = S.F32 if prec == "f32" else S.F64
    W, Ht, info = S.solve(S.dense(_t(A, dt)), _t(Wt, dt), S.params(lam=0.0, prec=p, max_outer=3))
    assert info["status"] == 0 and info["outer"] == 3
    assert np.array_equal(W.double().cpu().numpy(), Wt)
    assert np.array_equal(Ht.double().cpu().numpy(), Wt)
    assert info["res_WH"] == 0.0 and info["pg_norm"] == 0.0


@pytest.mark.parametrize("max_outer", [3, 100])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_start_check_leaves_outputs_untouched(S, prec, max_outer):
    """A start with a bad value in its last element (several copy pieces along) is refused
    whether the check is read with the results (short solves) or before them, the outputs
    keep their values, and the plan solves the next start as a fresh plan does."""
    dt = torch.float64 if prec == "f64" else torch.float32
    n, r = 1500, 7
    g = torch.Generator(device="cpu").manual_seed(3)
    W = torch.rand((n, r), generator=g, dtype=dt).to("cuda")
    A = W @ W.T
    A = 0.5 * (A + A.T)
    W0 = torch.rand((n, r), generator=g, dtype=dt).to("cuda")
    prm = S.params(lam=1.0, prec=S.prec_of(dt), max_outer=max_outer, check_every=1 << 30)
    with S.Plan(S.dense(A), r, prm) as pl:
        for bad, name in ((float("nan"), "E_NONFINITE"), (-1.0, "E_NEGATIVE")):
            Wb = W0.clone()
            Wb[-1, -1] = bad
            out = [torch.full_like(W0, 7.0) for _ in range(2)]
            with pytest.raises(S.SnmfError) as e:
                pl.solve(Wb, *out)
            assert e.value.name == name
            assert all(bool((o == 7.0).all()) for o in out)
        got = pl.solve(W0)
    with S.Plan(S.dense(A), r, prm) as pl:
        ref = pl.solve(W0)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


def test_batch_start_check_many_problems(S):
    """More problems than one copy launch takes: the first bad start decides the error."""
    n, r, k = 40, 3, 40
    g = torch.Generator(device="cpu").manual_seed(4)
    W = torch.rand((n, r), generator=g).to("cuda")
    A = W @ W.T
    A = 0.5 * (A + A.T)
    W0s = [torch.rand((2, n, r), generator=g).to("cuda") for _ in range(k)]
    with S.Batch([S.dense(A)] * k, [r] * k, S.params(lam=1.0, max_outer=2), 2) as b:
        Ws, Hs, infos, _ = b.solve(W0s)
        for i in (0, 33, k - 1):
            with S.Plan(S.dense(A), r, S.params(lam=1.0, max_outer=2, fuse_inner=0)) as pl:
                W, Ht, _ = pl.solve(W0s[i][1].contiguous())
            assert torch.equal(Ws[i][1], W) and torch.equal(Hs[i][1], Ht)
        for first, second, name in ((-1.0, float("inf"), "E_NEGATIVE"),
                                    (float("nan"), -1.0, "E_NONFINITE")):
            bad = [w.clone() for w in W0s]
            bad[34][1, 5, 1] = first
            bad[35][0, 0, 0] = second
            with pytest.raises(S.SnmfError) as e:
                b.solve(bad)
            assert e.value.name == name


def _plan_of_format(S, fmt, max_outer, **kw):
    n, r = 1500, 7
    g = torch.Generator(device="cpu").manual_seed(9)
    W0 = torch.rand((n, r), generator=g).to(DEV)
    prm = S.params(lam=1.0, max_outer=max_outer, check_every=1 << 30,
                   gamma=0.2 if fmt == "laplacian" else 0.0, **kw)
    if fmt == "lowrank":
        U = torch.linalg.qr(torch.rand((n, 12), generator=g))[0].contiguous().to(DEV)
        return S.Plan(S.lowrank(U, torch.linspace(9.0, 1.0, 12, dtype=torch.float64).to(DEV)), r,
                      prm), W0
    a = gen.random_symmetric_csr(n, 8.0, 5)
    L = None
    if fmt == "laplacian":
        L = S.csr_from_scipy(sp.csr_matrix(sp.eye(n) + sp.csr_matrix(a > 0) * -0.01), torch.float32)
    return S.Plan(S.csr_from_scipy(a, torch.float32), r, prm, L), W0


@pytest.mark.parametrize("fmt", ["csr", "laplacian", "lowrank"])
@pytest.mark.parametrize("max_outer", [3, 100])
def test_start_check_of_every_format(S, fmt, max_outer):
    """As above for the other formats of A and with the Laplacian term."""
    pl, W0 = _plan_of_format(S, fmt, max_outer)
    with pl:
        for bad, name in ((float("inf"), "E_NONFINITE"), (-1.0, "E_NEGATIVE")):
            Wb = W0.clone()
            Wb[700, 3] = bad
            out = [torch.full_like(W0, 7.0) for _ in range(2)]
            with pytest.raises(S.SnmfError) as e:
                pl.solve(Wb, *out)
            assert e.value.name == name
            assert all(bool((o == 7.0).all()) for o in out)
        got = pl.solve(W0)
    ref, _ = _plan_of_format(S, fmt, max_outer)
    with ref:
        ref = ref.solve(W0)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


def test_bad_start_ends_the_solve(S):
    """A start found bad by the check of a short solve ends it: its launches return at once
    (a negative entry alone would let the iteration run; both runs are the best of 8)."""
    n, r = 6000, 32
    g = torch.Generator(device="cpu").manual_seed(3)
    W = torch.rand((n, r), generator=g).to(DEV)
    A = W @ W.T
    W0 = torch.rand((n, r), generator=g).to(DEV)
    Wb = W0.clone()
    Wb[0, 0] = -1e-3

    def best(pl, w):
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            a = time.perf_counter()
            try:
                pl.solve(w, trace=False)
            except S.SnmfError as e:
                assert e.name == "E_NEGATIVE"
            t.append(time.perf_counter() - a)
        return min(t)

    with S.Plan(S.dense(0.5 * (A + A.T)), r, S.params(lam=1.0, max_outer=64)) as pl:
        good, bad = best(pl, W0), best(pl, Wb)
    assert bad <= 0.5 * good, (bad, good)


@pytest.mark.parametrize("kind", ["plan", "batch"])
def test_seconds_do_not_count_the_start_check(S, kind):
    """info.seconds and the trace's ticks start after the start is copied and checked: with and
    without the check (whose host wait takes some 20 us) the shortest of 40 tiny solves agree
    to 15%."""
    g = torch.Generator(device="cpu").manual_seed(1)
    W = torch.rand((40, 3), generator=g).to(DEV)
    A, W0 = S.dense(0.5 * (W @ W.T + (W @ W.T).T)), torch.rand((40, 3), generator=g).to(DEV)
    best = []
    for validate in (0, 1):
        prm = S.params(lam=1.0, max_outer=1 if kind == "batch" else 100, inner_iters=1,
                       validate=validate)
        if kind == "batch":
            with S.Batch([A], [3], prm, 1) as b:
                best.append(min(b.solve([W0[None].contiguous()])[2][0]["seconds"]
                                for _ in range(40)))
        else:
            with S.Plan(A, 3, prm) as pl:
                best.append(min(pl.solve(W0)[2]["trace"][0][5] for _ in range(40)))
    assert best[1] <= 1.15 * best[0], best


def test_plan_holds_no_direction_that_nothing_reads(S):
    """A plan of fused iterations on large arrays keeps seven n x r arrays (W, Ht, C, g, Z, the
    trial gradient, the product), and a half-step without fusing runs on it too."""
    n, r, ell = 200000, 32, 8
    g = torch.Generator(device="cpu").manual_seed(8)
    U = torch.linalg.qr(torch.rand((n, ell), generator=g))[0].contiguous().to(DEV)
    A = S.lowrank(U, torch.linspace(9.0, 1.0, ell, dtype=torch.float64).to(DEV))
    X = torch.rand((n, r), generator=g).to(DEV)
    S.Plan(A, 2, S.params(lam=1.0)).close()          # what the first use of the library allocates
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    with S.Plan(A, r, S.params(lam=1.0, max_outer=1)) as pl:
        used = free - torch.cuda.mem_get_info()[0]
        X1 = X.clone()
        pl.half_step(X1, X, False)
    assert used <= 7.6 * n * r * 4, used
    with S.Plan(A, r, S.params(lam=1.0, max_outer=1, fuse_inner=0)) as pl:
        X2 = X.clone()
        pl.half_step(X2, X, False)
    assert torch.equal(X1, X2)
