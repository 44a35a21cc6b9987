"""GPU parity: the HIP path (through the C ABI) against the FP64 oracle.

Integer outputs of the preparation are compared bit for bit; g', g'' and the
likelihood within the condition-scaled FP64 tolerance
    |dg'|  <= 1e-10 (sum_events |x_j| + sum_k d_k |G_k|)
    |dg''| <= 1e-10 sum_k d_k (|H_k| + G_k^2)
    |dL|   <= 1e-10 sum_k d_k |log S0_k|
(g' cancels near an optimum, so a plain relative bound would be meaningless
there; the rounding of a tree scan of N terms is ~ (log2 N + IPT) u).
"""
import numpy as np
import pytest

import gen
from oracle import ccd as occd, cv as ocv, km as okm, prep as oprep, risk, scan as oscan

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2204_08183_amd import survscan as ss  # noqa: E402

TOL = 1e-10
DEV = "cuda:0"


# ------------------------------------------------------------------ data
def make_case(model, n, p, seed, ties=0, density=0.05, valued=False, status=None,
              eta_shift=0.0):
    rng = np.random.default_rng(seed + 1000)
    d = gen.cox_data(seed, n, p, density) if model == "cox" else gen.fg_data(seed, n, p, density)
    y = d["y"]
    if ties:
        y = gen.force_ties(y, ties)
    st = d["status"].astype(np.int8)
    if status == "censored":
        st = np.zeros(n, np.int8)
    elif status == "events":
        st = np.ones(n, np.int8)
    vals = rng.normal(0.0, 1.0, d["rows"].size) if valued else None
    eta = rng.normal(0.0, 0.5, n) + eta_shift
    return {"y": y, "status": st, "col_ptr": d["col_ptr"], "rows": d["rows"], "vals": vals,
            "eta": eta, "n": n, "p": p}


def gpu_problem(model, c):
    prob = ss.Problem(model, c["y"], c["status"], c["col_ptr"], c["rows"], c["vals"], DEV)
    prob.set_eta(c["eta"])
    return prob


def xcol(c, j):
    return gen.dense_column(c["n"], c["col_ptr"], c["rows"], c["vals"], j)


def oracle_coord(model, c, j, prepared=None):
    x = xcol(c, j)
    if c["n"] <= 2000:
        r = risk.brute(model, c["y"], c["status"], c["eta"], x)
        ev = oprep.event_indicator(model, c["status"]) == 1
        return {"g1": r["g1"], "g2": r["g2"], "L": float(np.sum(np.log(r["S0"]))),
                "scale_g1": float(np.sum(np.abs(x[ev])) + np.sum(np.abs(r["G"]))),
                "scale_g2": float(np.sum(np.abs(r["H"]) + r["G"] ** 2)),
                "scale_L": float(np.sum(np.abs(np.log(r["S0"]))))}
    pr = prepared or oscan.Prepared(model, c["y"], c["status"])
    return pr.coordinate(c["eta"], x)


def assert_coord(got, want, what=""):
    g1, g2, L = (float(v) for v in got)
    assert abs(g1 - want["g1"]) <= TOL * want["scale_g1"] + 1e-300, (what, g1, want["g1"])
    assert abs(g2 - want["g2"]) <= TOL * want["scale_g2"] + 1e-300, (what, g2, want["g2"])
    assert abs(L - want["L"]) <= TOL * want["scale_L"] + 1e-300, (what, L, want["L"])


# ------------------------------------------------------------------ a0
PREP_CASES = [
    ("cox", 1, 3, 0, 0, 0.9), ("cox", 2, 3, 1, 0, 0.6), ("cox", 2049, 7, 2, 0, 0.05),
    ("cox", 6151, 9, 3, 40, 0.1), ("fg", 5000, 5, 4, 3, 0.3), ("fg", 3000, 6, 5, 0, 0.05),
    ("fg", 1, 2, 6, 0, 1.0),
]


@pytest.mark.parametrize("model,n,p,seed,ties,density", PREP_CASES)
@pytest.mark.parametrize("valued", [False, True])
def test_prepare_matches_oracle(model, n, p, seed, ties, density, valued):
    c = make_case(model, n, p, seed, ties, density, valued)
    prob = gpu_problem(model, c)
    order = oprep.order(c["y"])
    inv = np.empty_like(order)
    inv[order] = np.arange(n)
    ys = c["y"][order]
    ev = oprep.event_indicator(model, c["status"])[order]
    d = oprep.d_end(ys, ev)
    np.testing.assert_array_equal(prob.perm.cpu().numpy(), order)
    np.testing.assert_array_equal(prob.inv_perm.cpu().numpy(), inv)
    np.testing.assert_array_equal(prob.d32.cpu().numpy(), d)
    np.testing.assert_array_equal(prob.d8.cpu().numpy(), np.minimum(d, 255))
    rs, vs = oprep.csc_sorted_rows(c["col_ptr"], c["rows"], c["vals"], inv)
    nnz = c["rows"].size
    np.testing.assert_array_equal(prob.rows_sorted.cpu().numpy()[:nnz], rs)
    if valued:
        np.testing.assert_array_equal(prob.vals_sorted.cpu().numpy()[:nnz], vs)
    # chunk index: first offset in the column with position >= t * CHUNK
    cp = prob.chunk_ptr.cpu().numpy().reshape(p, prob.nchunk + 1)
    for j in range(p):
        a, b = c["col_ptr"][j], c["col_ptr"][j + 1]
        want = np.searchsorted(rs[a:b], np.arange(prob.nchunk + 1) * ss.CHUNK, side="left")
        np.testing.assert_array_equal(cp[j], want)
    # c_j = sum over events of x_ij
    ev_orig = oprep.event_indicator(model, c["status"])
    want_c = np.array([np.sum(xcol(c, j) * ev_orig) for j in range(p)])
    if valued:
        np.testing.assert_allclose(prob.c.cpu().numpy(), want_c, rtol=1e-13, atol=1e-12)
    else:
        np.testing.assert_array_equal(prob.c.cpu().numpy(), want_c)
    if model == "fg":
        t, v = okm.km_censoring(c["y"], c["status"])
        G = okm.km_eval(t, v, ys)
        np.testing.assert_allclose(prob.g_end.cpu().numpy(), G, rtol=1e-12, atol=0)
        W = np.where(c["status"][order] == 2, 1.0 / G, 0.0)
        np.testing.assert_allclose(prob.w_comp.cpu().numpy(), W, rtol=1e-12, atol=0)


# ------------------------------------------------------------------ a2 / a4
GH_CASES = [
    # n, p, seed, ties, density, valued, status, eta_shift
    (1, 2, 10, 0, 1.0, False, None, 0.0),
    (2, 2, 11, 0, 1.0, True, "events", 0.0),
    (2047, 4, 12, 0, 0.05, False, None, 0.0),
    (2048, 4, 13, 0, 0.05, True, None, 0.0),
    (2049, 4, 14, 0, 0.3, False, None, 0.0),
    (6151, 5, 15, 0, 0.05, False, None, 0.0),
    (6151, 5, 16, 25, 0.1, True, None, 0.0),
    (20000, 4, 17, 0, 0.05, False, None, 0.0),
    (20000, 3, 18, 3, 0.2, False, None, 0.0),     # runs with > 255 events
    (5000, 3, 19, 0, 0.05, False, "censored", 0.0),
    (5000, 3, 20, 0, 0.05, True, "events", 0.0),
    (9000, 3, 21, 0, 1.0, False, None, 0.0),      # dense column
    (70001, 3, 26, 30, 1.0, True, None, 0.0),     # dense valued, ragged last tile
    (9000, 3, 22, 0, 0.05, False, None, 600.0),   # large eta, FP64 range
    (100000, 3, 23, 50, 0.05, True, None, 0.0),
]


@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n,p,seed,ties,density,valued,status,shift", GH_CASES)
def test_grad_hess_matches_oracle(model, n, p, seed, ties, density, valued, status, shift):
    c = make_case(model, n, p, seed, ties, density, valued, status, shift)
    prob = gpu_problem(model, c)
    pr = oscan.Prepared(model, c["y"], c["status"]) if n > 2000 else None
    for j in range(p):
        got = prob.grad_hess(j).cpu().numpy()
        assert_coord(got, oracle_coord(model, c, j, pr), (model, n, j))
    assert prob.workspace_error() == 0


# Above 1,572,864 positions the fused kernel runs tiles of 4096 positions
# (16 per thread).  Tie runs of every length cross those tile boundaries, and
# with 1500 distinct times (about 1333 subjects per run) nearly every run holds
# more than 255 events under both models (Fine-Gray counts status 1 only,
# about a quarter of the subjects), so the event
# counts of a run end take the 32-bit escape.
LARGE_TIE_CASES = [
    # n, p, seed, ties, density, valued
    (2_000_003, 3, 24, 1500, 0.05, False),
    (1_900_000, 2, 25, 400_000, 0.3, True),
]


@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n,p,seed,ties,density,valued", LARGE_TIE_CASES)
def test_grad_hess_large_tiles_with_ties(model, n, p, seed, ties, density, valued):
    c = make_case(model, n, p, seed, ties, density, valued)
    prob = gpu_problem(model, c)
    d32 = prob.d32.cpu().numpy()
    if ties == 1500:
        assert np.count_nonzero(d32 >= 255) > 100
    pr = oscan.Prepared(model, c["y"], c["status"])
    for j in range(p):
        got = prob.grad_hess(j).cpu().numpy()
        assert_coord(got, oracle_coord(model, c, j, pr), (model, n, j))
    assert prob.workspace_error() == 0


@pytest.mark.parametrize("model", ["cox", "fg"])
def test_empty_column(model):
    c = make_case(model, 3000, 2, 30, 0, 0.05)
    c["col_ptr"] = np.array([0, 0, c["col_ptr"][1]], dtype=np.int64)
    c["rows"] = c["rows"][: c["col_ptr"][2]]
    prob = gpu_problem(model, c)
    got = prob.grad_hess(0).cpu().numpy()
    want = oracle_coord(model, c, 0)
    assert got[0] == 0.0 and got[1] == 0.0
    assert abs(got[2] - want["L"]) <= TOL * want["scale_L"]


@pytest.mark.parametrize("model", ["cox", "fg"])
def test_repeated_calls_reuse_workspace(model):
    """The launch counters reset themselves: 50 calls in a row agree."""
    c = make_case(model, 30000, 2, 31, 0, 0.05)
    prob = gpu_problem(model, c)
    outs = torch.stack([prob.grad_hess(1, out=torch.empty(3, dtype=torch.float64,
                                                           device=DEV)) for _ in range(50)])
    want = oracle_coord(model, c, 1)
    for row in outs.cpu().numpy():
        assert_coord(row, want)
    assert prob.workspace_error() == 0


# ------------------------------------------------------------------ likelihood
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n,ties", [(1500, 0), (40000, 30)])
def test_loglik_matches_oracle(model, n, ties):
    c = make_case(model, n, 6, 40, ties, 0.1)
    rng = np.random.default_rng(1)
    beta = rng.normal(0, 0.3, 6)
    c["eta"] = gen.linear_predictor(n, c["col_ptr"], c["rows"], None, beta)
    prob = gpu_problem(model, c)
    got = float(prob.loglik(beta).cpu().numpy()[0])
    if n <= 2000:
        want = risk.loglik(model, c["y"], c["status"], c["eta"])
        scale = abs(want) * 1.0
    else:
        r = oscan.Prepared(model, c["y"], c["status"]).coordinate(c["eta"], np.zeros(n))
        want, scale = r["loglik"], r["scale_L"] + abs(r["loglik"])
    assert abs(got - want) <= TOL * scale


@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("penalty,lam", [("none", 0.0), ("l1", 1.5), ("l2", 0.7)])
def test_objective_matches_oracle(model, penalty, lam):
    """ss_objective: l + pi on the device against the oracle's likelihood
    (O(N^2) definition) and penalty (Sec. 2.3)."""
    n, p = 1800, 6
    c = make_case(model, n, p, 41, 20, 0.1, valued=True)
    rng = np.random.default_rng(2)
    beta = rng.normal(0, 0.4, p)
    beta[2] = 0.0
    c["eta"] = gen.linear_predictor(n, c["col_ptr"], c["rows"], c["vals"], beta)
    prob = gpu_problem(model, c)
    prob.beta.copy_(torch.as_tensor(beta))
    got = prob.objective(penalty, lam).cpu().numpy()
    pen = {"none": occd.PENALTY_NONE, "l1": occd.PENALTY_L1, "l2": occd.PENALTY_L2}[penalty]
    want_l = float(risk.loglik(model, c["y"], c["status"], c["eta"]))
    want_pi = occd.penalty_value(beta, pen, lam)
    r = risk.brute(model, c["y"], c["status"], c["eta"], np.zeros(n))
    scale = float(np.sum(np.abs(np.log(r["S0"])))) + abs(want_l) + abs(want_pi)
    assert abs(got[1] - want_l) <= TOL * scale, (got[1], want_l)
    assert abs(got[2] - want_pi) <= 1e-14 * (abs(want_pi) + 1.0), (got[2], want_pi)
    assert abs(got[0] - (want_l + want_pi)) <= TOL * scale
    assert prob.workspace_error() == 0


def test_cv_select_by_hand():
    """ss_cv_select: per-strength means of the held-out scores (the odd
    entries of each row) and the first strength with the largest mean."""
    lib = ss.load()
    reps = 3
    # rows: (train, held-out) pairs per replicate; held-out means -2, -1, -1, NaN
    table = np.array([[9.0, -1.0, 9.0, -2.0, 9.0, -3.0],
                      [0.0, -1.0, 0.0, -1.0, 0.0, -1.0],
                      [5.0, -0.5, 5.0, -1.5, 5.0, -1.0],
                      [0.0, float("nan"), 0.0, 1.0, 0.0, 1.0]])
    t = torch.as_tensor(table, device=DEV)
    mean = torch.empty(4, dtype=torch.float64, device=DEV)
    best = torch.full((1,), 7, dtype=torch.int32, device=DEV)
    s = ss._stream(torch.device(DEV))
    assert lib.ss_cv_select(4, reps, ss._p(t), ss._p(mean), ss._p(best), s) == ss.SS_OK
    m = mean.cpu().numpy()
    np.testing.assert_array_equal(m[:3], [-2.0, -1.0, -1.0])
    assert np.isnan(m[3])
    assert int(best.cpu()[0]) == 1


# ------------------------------------------------------------------ a3 + a1
@pytest.mark.parametrize("penalty,lam,g1,g2,b,dj", [
    ("none", 0.0, 3.0, -2.0, 0.1, 1.0), ("none", 0.0, 3.0, -2.0, 0.1, 0.25),
    ("l2", 0.5, 1.0, -4.0, 0.3, 1.0), ("l1", 1.0, 3.0, -2.0, 0.0, 5.0),
    ("l1", 1.0, -3.0, -2.0, 0.0, 5.0), ("l1", 1.0, 0.2, -2.0, 0.0, 5.0),
    ("l1", 1.0, -5.0, -2.0, 0.5, 5.0), ("l1", 1.0, 1.5, -2.0, -0.2, 5.0),
    ("none", 0.0, 1.0, 0.0, 0.0, 1.0),
])
def test_ccd_update_matches_oracle(penalty, lam, g1, g2, b, dj):
    c = make_case("cox", 5000, 3, 50, 0, 0.1, valued=True)
    prob = gpu_problem("cox", c)
    j = 1
    prob.beta[j] = b
    prob.delta[j] = dj
    g12 = torch.tensor([g1, g2, 0.0], dtype=torch.float64, device=DEV)
    eta0 = prob.eta.cpu().numpy().copy()
    prob.ccd_update(j, g12, penalty, lam)
    pen = {"none": occd.PENALTY_NONE, "l1": occd.PENALTY_L1, "l2": occd.PENALTY_L2}[penalty]
    nb, nd, step = occd.update(g1, g2, b, dj, pen, lam)
    assert float(prob.beta[j]) == nb
    assert float(prob.delta[j]) == nd
    assert float(prob.steps[j]) == step
    x_s = xcol(c, j)[prob.perm.cpu().numpy()]
    want_eta = eta0 + x_s * step
    np.testing.assert_allclose(prob.eta.cpu().numpy(), want_eta, rtol=1e-15, atol=1e-15)
    np.testing.assert_allclose(prob.e.cpu().numpy(), np.exp(want_eta), rtol=1e-14)


# ------------------------------------------------------------------ fused sweep
def oracle_sweeps(model, c, penalty, lam, sweeps):
    """The oracle's CCD loop (oracle.cv.ccd_sweeps, pinned on the CPU) from
    beta = 0 at the case's eta."""
    return ocv.ccd_sweeps(model, c["y"], c["status"], c["col_ptr"], c["rows"], c["vals"],
                          c["eta"], penalty, lam, sweeps)


SWEEP_PATHS = ["persistent", "launch"]


def _sweep_env(monkeypatch, path):
    if path == "launch":
        monkeypatch.setenv("SURVSCAN_SWEEP", "launch")
    else:
        monkeypatch.delenv("SURVSCAN_SWEEP", raising=False)


@pytest.mark.parametrize("path", SWEEP_PATHS)
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("penalty,lam", [(occd.PENALTY_L1, 2.0), (occd.PENALTY_L2, 1.0),
                                         (occd.PENALTY_NONE, 0.0)])
def test_sweep_matches_oracle_ccd(model, penalty, lam, path, monkeypatch):
    _sweep_env(monkeypatch, path)
    c = make_case(model, 7000, 10, 60, 0, 0.2)
    c["eta"] = np.zeros(c["n"])
    prob = gpu_problem(model, c)
    name = {occd.PENALTY_NONE: "none", occd.PENALTY_L1: "l1", occd.PENALTY_L2: "l2"}[penalty]
    g12 = torch.zeros(3 * c["p"], dtype=torch.float64, device=DEV)
    beta, delta, eta, hist = oracle_sweeps(model, c, penalty, lam, 2)
    for s in range(2):
        prob.sweep(name, lam, g12_out=g12)
        got = g12.cpu().numpy().reshape(-1, 3)
        for j in range(c["p"]):
            g1, g2, s1, s2 = hist[s * c["p"] + j]
            assert abs(got[j, 0] - g1) <= 1e-9 * s1, (s, j)
            assert abs(got[j, 1] - g2) <= 1e-9 * s2, (s, j)
    np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-8, atol=1e-12)
    np.testing.assert_allclose(prob.delta.cpu().numpy(), delta, rtol=1e-8, atol=1e-12)
    order = prob.perm.cpu().numpy()
    np.testing.assert_allclose(prob.eta.cpu().numpy(), eta[order], rtol=1e-8, atol=1e-10)
    np.testing.assert_allclose(prob.e.cpu().numpy(), np.exp(eta[order]), rtol=1e-8)
    assert prob.workspace_error() == 0


@pytest.mark.parametrize("path", SWEEP_PATHS)
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n,p,ties,valued", [
    (1_000_000, 6, 0, False),     # the benchmark size: 489 segments of 2048
    (2_500_003, 4, 0, True),      # segments of 8192, ragged last segment
    (300_001, 5, 40, False),      # tie runs across segment boundaries
    (4_300_000, 3, 0, False),     # above the persistent limit: launch per coordinate
    (2_000_003, 3, 3000, False),  # 4096-position tiles, runs of 255+ events
])
def test_sweep_large(model, n, p, ties, valued, path, monkeypatch):
    _sweep_env(monkeypatch, path)
    c = make_case(model, n, p, 70, ties, 0.05, valued)
    c["eta"] = np.zeros(n)
    prob = gpu_problem(model, c)
    lam = 1.0
    g12 = torch.zeros(3 * p, dtype=torch.float64, device=DEV)
    beta, delta, eta, hist = oracle_sweeps(model, c, occd.PENALTY_L1, lam, 1)
    prob.sweep("l1", lam, g12_out=g12)
    got = g12.cpu().numpy().reshape(-1, 3)
    for j in range(p):
        g1, g2, s1, s2 = hist[j]
        assert abs(got[j, 0] - g1) <= 1e-10 * s1, (j, got[j, 0], g1)
        assert abs(got[j, 1] - g2) <= 1e-10 * s2, (j, got[j, 1], g2)
    np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-9, atol=1e-13)
    order = prob.perm.cpu().numpy()
    np.testing.assert_allclose(prob.eta.cpu().numpy(), eta[order], rtol=1e-9, atol=1e-12)
    assert prob.workspace_error() == 0


@pytest.mark.parametrize("model", ["cox", "fg"])
def test_sweep_deterministic_and_consistent(model, monkeypatch):
    """The persistent sweep adds every partial in a fixed order: two runs
    from the same state agree bit for bit, and grad_hess afterwards sees the
    e the sweep left behind."""
    monkeypatch.delenv("SURVSCAN_SWEEP", raising=False)
    c = make_case(model, 200_000, 8, 80, 0, 0.05)
    c["eta"] = np.zeros(c["n"])
    outs = []
    for _ in range(2):
        prob = gpu_problem(model, c)
        g12 = torch.zeros(3 * c["p"], dtype=torch.float64, device=DEV)
        prob.sweep("l1", 0.5, g12_out=g12)
        prob.sweep("l1", 0.5, g12_out=g12)
        outs.append((g12.cpu().numpy().copy(), prob.beta.cpu().numpy().copy(),
                     prob.e.cpu().numpy().copy()))
        # e is consistent with eta after the sweep
        np.testing.assert_allclose(prob.e.cpu().numpy(), np.exp(prob.eta.cpu().numpy()),
                                   rtol=1e-14)
        assert prob.workspace_error() == 0
    for a_, b_ in zip(outs[0], outs[1]):
        np.testing.assert_array_equal(a_, b_)
    # without g12_out the sweep does not form or exchange sum d log S0 (a
    # kernel of its own): the same coefficients and e, bit for bit
    prob = gpu_problem(model, c)
    prob.sweep("l1", 0.5)
    prob.sweep("l1", 0.5)
    np.testing.assert_array_equal(prob.beta.cpu().numpy(), outs[0][1])
    np.testing.assert_array_equal(prob.e.cpu().numpy(), outs[0][2])
    assert prob.workspace_error() == 0


@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("penalty,lam", [("l1", 4.0), ("l2", 0.5)])
def test_fit_reaches_kkt(model, penalty, lam):
    """Sweeps to convergence satisfy the optimality conditions of the
    penalised objective: l1, |g'_j| <= gamma where beta_j = 0 and
    g'_j = gamma sgn(beta_j) elsewhere; l2, g'_j = beta_j / tau.  The
    coefficients also match the oracle's coordinate descent run for the
    same number of sweeps."""
    c = make_case(model, 6000, 8, 90, 0, 0.2)
    c["eta"] = np.zeros(c["n"])
    prob = gpu_problem(model, c)
    sweeps = prob.fit(penalty, lam, max_sweeps=300, tol=1e-15)
    assert sweeps < 300
    assert prob.workspace_error() == 0
    beta = prob.beta.cpu().numpy()
    pen = {"l1": occd.PENALTY_L1, "l2": occd.PENALTY_L2}[penalty]
    b_or, _, _, _ = oracle_sweeps(model, c, pen, lam, sweeps)
    np.testing.assert_allclose(beta, b_or, rtol=1e-7, atol=1e-10)
    g = np.array([prob.grad_hess(j).cpu().numpy() for j in range(c["p"])])
    g1, g2 = g[:, 0], g[:, 1]
    # what is left of a Newton step at the optimum: at most 1e-6
    if penalty == "l1":
        assert np.any(beta == 0.0) and np.any(beta != 0.0)
        zero = beta == 0.0
        assert np.all(np.abs(g1[zero]) - lam <= 1e-6 * np.abs(g2[zero]))
        assert np.all(np.abs(g1[~zero] - lam * np.sign(beta[~zero]))
                      <= 1e-6 * np.abs(g2[~zero]))
    else:
        assert np.all(np.abs(g1 - beta / lam) <= 1e-6 * (np.abs(g2) + 1.0 / lam))


@pytest.mark.parametrize("name", ["cox_hand", "cox_ties_hand", "fg_hand"])
def test_hand_examples(name):
    """The HIP path on the hand-derived examples of tests/golden."""
    import golden
    g = golden.load(name)
    n = len(g["y"])
    x = np.array(g["x"])
    rows = np.nonzero(x)[0].astype(np.int32)
    prob = ss.Problem(g["model"], g["y"], np.array(g["status"], np.int8),
                      np.array([0, rows.size], np.int64), rows, None, DEV)
    prob.set_eta(np.array(g["eta"]))
    got = prob.grad_hess(0).cpu().numpy()
    assert got[0] == pytest.approx(g["g1"], rel=1e-14, abs=1e-15)
    assert got[1] == pytest.approx(g["g2"], rel=1e-14, abs=1e-15)
    ll = float(prob.loglik().cpu()[0])
    assert ll == pytest.approx(g["loglik"], rel=1e-14, abs=1e-15)
    assert n == prob.n


# The design's ordering: a column is one LDS bitmap up to 2^20 positions, cut
# into windows above that and where few long columns would leave the chip
# idle; pieces with few entries for their window are sorted in LDS instead
# (at most 1024 of them, fewer than one per 512 positions).
DESIGN_CASES = [
    # n, entries per column
    (131_072, [0, 1, 255, 256, 257, 131_072]),        # the line between the two, W / 512
    (131_073, [255, 256, 257, 131_073, 131_072]),     # the larger workgroup; a full column
    (1_048_576, [1023, 1024, 1025, 2048, 60_000]),    # the largest single window
    (1_048_577, [0, 1, 1024, 1025, 70_000]),          # two windows, the last one position
    (2_100_000, [900_000, 300, 2_100_000]),           # windows cut further, nearly full
    (40_000, [20_000, 40_000]),                       # short columns cut further
]


@pytest.mark.parametrize("valued", [False, True])
@pytest.mark.parametrize("n,counts", DESIGN_CASES)
def test_design_ordering(n, counts, valued):
    rng = np.random.default_rng(n)
    y = rng.random(n)
    status = (rng.random(n) < 0.5).astype(np.int8)
    rows = np.concatenate([rng.permutation(n)[:m] for m in counts]).astype(np.int32)
    vals = rng.uniform(1.0, 2.0, rows.size) if valued else None
    col_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    prob = ss.Problem("cox", y, status, col_ptr, rows, vals)
    order = np.argsort(-y, kind="stable")
    inv = np.empty_like(order)
    inv[order] = np.arange(n)
    rs, vs = oprep.csc_sorted_rows(col_ptr, rows, vals, inv)
    np.testing.assert_array_equal(prob.rows_sorted.cpu().numpy()[:rs.size], rs)
    if valued:
        np.testing.assert_array_equal(prob.vals_sorted.cpu().numpy()[:rs.size], vs)
    cp = prob.chunk_ptr.cpu().numpy().reshape(len(counts), prob.nchunk + 1)
    edges = np.arange(prob.nchunk + 1) * ss.CHUNK
    got_c = prob.c.cpu().numpy()
    for j in range(len(counts)):
        a, b = col_ptr[j], col_ptr[j + 1]
        np.testing.assert_array_equal(cp[j], np.searchsorted(rs[a:b], edges, side="left"))
        x = np.ones(b - a) if vals is None else vals[a:b]
        want = float(np.sum(x * status[rows[a:b]]))
        # fixed-order sums of at most 2^21 terms in [1, 2]
        assert abs(got_c[j] - want) <= (2.0 ** -31 * want if valued else 0.0), j


def _times(kind, n, rng):
    if kind == "whole":        # few bits vary: all of them are ordered
        return np.ceil(rng.random(n) * 300)
    if kind == "continuous":   # small groups agree in the bits ordered
        return rng.standard_normal(n)
    if kind == "one":          # nothing varies
        return np.full(n, 2.5)
    # one far time and the others close together: groups of 32 records and one
    # of equal ones ("close"), or all records in one ("closest"), agree in the
    # bits ordered
    y = 1e6 + rng.permutation(n) * (2.0 ** -7 if kind == "close" else 2.0 ** -30)
    y[rng.integers(0, n, n // 8)] = 1e6 - 2.0 ** -3  # equal ones
    y[n // 2] = 0.25
    if kind == "signed":
        y = np.where(rng.random(n) < 0.5, y - 1e6, 1e6 - y)
        y[:2] = np.array([0.0, -0.0])[:n]
    return y


@pytest.mark.parametrize("kind", ["whole", "continuous", "one", "close", "closest", "signed"])
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 2047, 2049, 4096, 4097, 300_001, 1_048_577])
def test_time_ordering(n, model, kind):
    """Order, events at run ends and weights: one tile of the sort and the
    scans to many, and every way the bits of the times can be ordered."""
    rng = np.random.default_rng(n)
    y = _times(kind, n, rng)
    status = rng.integers(0, 3 if model == "fg" else 2, n).astype(np.int8)
    prob = ss.Problem(model, y, status, np.array([0, 1]), np.array([0], dtype=np.int32))
    order = np.argsort(-y, kind="stable")
    np.testing.assert_array_equal(prob.perm.cpu().numpy(), order)
    inv = np.empty_like(order)
    inv[order] = np.arange(n)
    np.testing.assert_array_equal(prob.inv_perm.cpu().numpy(), inv)
    ys, st = y[order], status[order]
    end = np.append(ys[1:] != ys[:-1], True)
    start_of = np.concatenate([[0], np.cumsum(end)[:-1]])  # run of each position
    d = np.bincount(start_of, st == 1 if model == "fg" else st != 0)
    want = np.where(end, d[start_of], 0).astype(np.int64)
    np.testing.assert_array_equal(prob.d32.cpu().numpy(), want)
    np.testing.assert_array_equal(prob.d8.cpu().numpy()[:n], np.minimum(want, 255))
    if model == "fg":
        cens = np.bincount(start_of, st == 0)
        fac = np.where(end, 1.0 - cens[start_of] / np.arange(1, n + 1), 1.0)
        g = np.cumprod(fac[::-1].astype(np.longdouble))[::-1]
        # at most n roundings of 2^-53 each, in either order of the product
        tol = (n + 2) * 2.0 ** -52
        np.testing.assert_allclose(prob.g_end.cpu().numpy(), g.astype(np.float64), rtol=tol,
                                   atol=1e-300)
        with np.errstate(divide="ignore"):
            w = np.where(st == 2, 1.0 / prob.g_end.cpu().numpy(), 0.0)
        np.testing.assert_array_equal(prob.w_comp.cpu().numpy(), w)


# more tiles than a workgroup adds up itself: of the run and weight scans, of
# the times that order 40 bits, of the digit counts; a record without status
@pytest.mark.parametrize("n", [4_300_000, 8_400_000, 67_200_000, 2**30 + 5])
def test_time_ordering_large(n):
    if torch.cuda.mem_get_info()[0] < 140 * n:
        pytest.skip("needs %.0f GB" % (140e-9 * n))
    g = torch.Generator(device="cuda").manual_seed(n)
    y = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    y[::7] = torch.round(y[::7] * 4096) / 4096
    status = torch.randint(0, 3, (n,), dtype=torch.int8, device="cuda", generator=g)
    prob = ss.Problem("fg", y, status, np.array([0, 1]), np.array([0], dtype=np.int32))
    ys, order = torch.sort(y, descending=True, stable=True)
    assert torch.equal(prob.perm.long(), order)
    assert torch.equal(prob.inv_perm[order].long(), torch.arange(n, device="cuda"))
    st = status[order]
    end = torch.ones(n, dtype=torch.bool, device="cuda")
    end[:-1] = ys[1:] != ys[:-1]
    last = torch.nonzero(end).flatten()

    def at_ends(mark):
        upto = torch.cumsum(mark.long(), 0)[last]
        return torch.diff(upto, prepend=upto.new_zeros(1))

    want = torch.zeros(n, dtype=torch.int32, device="cuda")
    want[last] = at_ends(st == 1).int()
    assert torch.equal(prob.d32, want)
    fac = torch.ones(n, dtype=torch.float64, device="cuda")
    fac[last] = 1.0 - at_ends(st == 0).double() / (last + 1).double()
    km = torch.cumprod(fac.flip(0), 0).flip(0)
    # at most n roundings of 2^-53 each, on both sides
    assert torch.allclose(prob.g_end, km, rtol=(n + 2) * 2.0 ** -52, atol=1e-300)


@pytest.mark.parametrize("n,m", [(3000, 40), (300_000, 30), (300_000, 2000), (2_100_000, 50_000)])
def test_design_errors(n, m):
    """A duplicate row and a row out of range are still refused, on every
    path of the ordering."""
    rng = np.random.default_rng(m)
    rows = rng.permutation(n)[:m].astype(np.int32)
    y, status = rng.random(n), np.ones(n, dtype=np.int8)
    ptr = np.array([0, m], dtype=np.int64)
    for bad in (int(rows[0]), n, -1):
        r = rows.copy()
        r[m - 1] = bad
        with pytest.raises(ss.SurvScanError):
            ss.Problem("cox", y, status, ptr, r)


# Both sides of every line of the persistent sweep's built-in shapes: one
# workgroup up to 4096 (valued: 2048) positions, segments of 1024 up to 2^18
# (Fine-Gray 0/1: 2^17), of 2048 up to 2^19, of 4096 above; and more segments
# than a gather has threads.
SHAPE_SIZES = [1023, 1024, 1025, 2048, 2049, 4096, 4097, 131_072, 131_073, 262_145, 524_289]


@pytest.mark.parametrize("valued", [False, True])
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n", SHAPE_SIZES)
def test_sweep_shapes(n, model, valued):
    p = 7
    c = make_case(model, n, p, n, 0, 0.05 if not valued else 0.4, valued)
    c["y"] = np.ceil(c["y"] * n / 2)  # tie runs
    c["eta"] = np.zeros(n)
    prob = gpu_problem(model, c)
    g12 = torch.zeros(3 * p, dtype=torch.float64, device=DEV)
    beta, delta, eta, hist = oracle_sweeps(model, c, occd.PENALTY_L2, 1.0, 1)
    prob.sweep("l2", 1.0, g12_out=g12)
    got = g12.cpu().numpy().reshape(-1, 3)
    for j in range(p):
        g1, g2, s1, s2 = hist[j]
        assert abs(got[j, 0] - g1) <= 1e-10 * s1, (j, got[j, 0], g1)
        assert abs(got[j, 1] - g2) <= 1e-10 * s2, (j, got[j, 1], g2)
    np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-9, atol=1e-13)
    order = prob.perm.cpu().numpy()
    np.testing.assert_allclose(prob.eta.cpu().numpy(), eta[order], rtol=1e-9, atol=1e-12)
    np.testing.assert_allclose(prob.e.cpu().numpy(), np.exp(prob.eta.cpu().numpy()), rtol=1e-14)
    # a second run from the same state: bit for bit
    first = prob.beta.clone(), prob.e.clone()
    prob.set_beta(torch.zeros(p), np.zeros(n))
    prob.reset_trust()
    prob.sweep("l2", 1.0)
    assert torch.equal(prob.beta, first[0]) and torch.equal(prob.e, first[1])
    # single-coordinate and split sweeps continue from the state left behind
    prob.set_beta(torch.zeros(p), np.zeros(n))
    prob.reset_trust()
    prob.sweep("l2", 1.0, j_begin=0, j_end=1)
    prob.sweep("l2", 1.0, j_begin=1, j_end=3)
    prob.sweep("l2", 1.0, j_begin=3, j_end=p)
    np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-9, atol=1e-13)
    assert prob.workspace_error() == 0


# The per-coordinate launches of a 0/1 sweep take a tile's prefix from the
# tile sums the launch before left (tiles of 2048 positions in groups of 64)
# and bring eta up to date at the end, 64 columns and 64 non-zeros of a chunk
# at a time: around one tile, one, two and three groups.
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n,p,density", [
    (1000, 3, 0.2), (2048, 65, 0.1), (2049, 64, 0.5), (131_072, 5, 0.05), (131_073, 70, 0.1),
    (262_145, 4, 0.05)])
def test_sweep_launches_tile_sums(model, n, p, density, monkeypatch):
    _sweep_env(monkeypatch, "launch")
    c = make_case(model, n, p, 90 + p, 0, density)
    c["y"] = np.ceil(c["y"] * n)  # some tie runs
    c["eta"] = np.zeros(n)
    prob = gpu_problem(model, c)
    g12 = torch.zeros(3 * p, dtype=torch.float64, device=DEV)
    beta, delta, eta, hist = oracle_sweeps(model, c, occd.PENALTY_L2, 1.0, 1)
    for upto in (None, p):  # with and without the per-coordinate output
        prob.set_beta(torch.zeros(p), np.zeros(n))
        prob.reset_trust()
        prob.sweep("l2", 1.0, g12_out=g12 if upto else None)
        np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-9, atol=1e-13)
    got = g12.cpu().numpy().reshape(-1, 3)
    for j in range(p):
        g1, g2, s1, s2 = hist[j]
        assert abs(got[j, 0] - g1) <= 1e-10 * s1, (j, got[j, 0], g1)
        assert abs(got[j, 1] - g2) <= 1e-10 * s2, (j, got[j, 1], g2)
    order = prob.perm.cpu().numpy()
    np.testing.assert_allclose(prob.eta.cpu().numpy(), eta[order], rtol=1e-9, atol=1e-12)
    np.testing.assert_allclose(prob.e.cpu().numpy(), np.exp(prob.eta.cpu().numpy()), rtol=1e-14)
    # parts of a sweep, of one and more coordinates, continue from the state
    prob.set_beta(torch.zeros(p), np.zeros(n))
    prob.reset_trust()
    for a, b in ((0, 1), (1, 3), (3, p)):
        prob.sweep("l2", 1.0, j_begin=a, j_end=b)
    np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-9, atol=1e-13)
    assert prob.workspace_error() == 0


# The latest subjects, censored, with an e that underflows to 0 (eta = -800)
# or to a subnormal without a finite reciprocal (eta = -720): no run ends
# there, and nothing of them may reach the sums.  One workgroup of each shape,
# and several.
@pytest.mark.parametrize("path", SWEEP_PATHS)
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n", [900, 1800, 3000, 7000])
def test_sweep_leading_underflow(n, model, path, monkeypatch):
    _sweep_env(monkeypatch, path)
    p = 6
    c = make_case(model, n, p, 130, 0, 0.1)
    latest = np.argsort(-c["y"], kind="stable")[:40]
    c["status"][latest] = 0
    c["eta"] = np.random.default_rng(131).normal(0.0, 0.5, n)
    c["eta"][latest[:20]] = -800.0
    c["eta"][latest[20:]] = -720.0
    prob = gpu_problem(model, c)
    g12 = torch.zeros(3 * p, dtype=torch.float64, device=DEV)
    beta, delta, eta, hist = oracle_sweeps(model, c, occd.PENALTY_L2, 1.0, 1)
    for out in (None, g12):  # without and with the per-coordinate output
        prob.set_beta(torch.zeros(p), c["eta"])
        prob.reset_trust()
        prob.sweep("l2", 1.0, g12_out=out)
        np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-9, atol=1e-13)
    got = g12.cpu().numpy().reshape(-1, 3)
    for j in range(p):
        g1, g2, s1, s2 = hist[j]
        assert abs(got[j, 0] - g1) <= 1e-10 * s1, (j, got[j, 0], g1)
        assert abs(got[j, 1] - g2) <= 1e-10 * s2, (j, got[j, 1], g2)
    assert prob.workspace_error() == 0


def _check_history(prob, c, g12, hist, tol=1e-10):
    got = g12.cpu().numpy().reshape(-1, 3)
    for j in range(c["p"]):
        g1, g2, s1, s2 = hist[j]
        assert abs(got[j, 0] - g1) <= tol * s1, (j, got[j, 0], g1)
        assert abs(got[j, 1] - g2) <= tol * s2, (j, got[j, 1], g2)
    assert prob.workspace_error() == 0


def _columns(n, cols):
    ptr = np.concatenate([[0], np.cumsum([len(r) for r in cols])]).astype(np.int64)
    return ptr, np.concatenate(cols).astype(np.int32)


# Sweeps by launches take e = exp(eta) afresh at every update: an e that has
# underflowed to 0 (eta = -800) comes back once eta does, 100 a coordinate,
# and counts in the coordinates after it.
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n", [1500, 9000])
def test_sweep_launches_bring_e_back(n, model, monkeypatch):
    _sweep_env(monkeypatch, "launch")
    c = make_case(model, n, 3, 140, 0, 0.1)
    order = np.argsort(-c["y"], kind="stable")
    who = int(order[3])                          # early: large in many risk sets
    c["status"][order[:12]] = 1
    rng = np.random.default_rng(141)
    cols = [np.array([who])] * 8 + [rng.choice(n, n // 10, replace=False) for _ in range(4)]
    cols[9] = np.union1d(cols[9], [who])
    c["col_ptr"], c["rows"] = _columns(n, cols)
    c["p"] = p = len(cols)
    c["eta"] = rng.normal(0.0, 0.5, n)
    c["eta"][who] = -800.0
    prob = gpu_problem(model, c)
    prob.delta.fill_(200.0)
    g12 = torch.zeros(3 * p, dtype=torch.float64, device=DEV)
    beta, delta, eta, hist = ocv.ccd_sweeps(model, c["y"], c["status"], c["col_ptr"], c["rows"],
                                            None, c["eta"], occd.PENALTY_L2, 100.0, 1,
                                            delta=np.full(p, 200.0))
    assert eta[who] > -5.0                       # it did come back
    prob.sweep("l2", 100.0, g12_out=g12)
    _check_history(prob, c, g12, hist)
    np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-9, atol=1e-12)


# A step of -20 on a column that covers the first half of the positions: the
# prefixes after it are e^-20 of those before, and as accurate.
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n", [20_000, 300_001])
def test_sweep_launches_large_negative_step(n, model, monkeypatch):
    _sweep_env(monkeypatch, "launch")
    c = make_case(model, n, 3, 150, 0, 0.1)
    order = np.argsort(-c["y"], kind="stable")
    rng = np.random.default_rng(151)
    half = order[: n // 2]
    c["eta"] = rng.normal(0.0, 0.3, n)
    c["eta"][order[n // 2:]] -= 8.0
    cols = [np.sort(half)] + [np.sort(rng.choice(n, n // 20, replace=False)) for _ in range(3)]
    c["col_ptr"], c["rows"] = _columns(n, cols)
    c["p"] = p = len(cols)
    prob = gpu_problem(model, c)
    prob.delta.fill_(20.0)
    g12 = torch.zeros(3 * p, dtype=torch.float64, device=DEV)
    beta, delta, eta, hist = ocv.ccd_sweeps(model, c["y"], c["status"], c["col_ptr"], c["rows"],
                                            None, c["eta"], occd.PENALTY_NONE, 0.0, 1,
                                            delta=np.full(p, 20.0))
    assert beta[0] == -20.0
    prob.sweep("none", 0.0, g12_out=g12)
    _check_history(prob, c, g12, hist)
    np.testing.assert_allclose(prob.beta.cpu().numpy(), beta, rtol=1e-9, atol=1e-12)


# Times in groups of exactly m that agree in the bits the sort orders and
# differ below (some of them equal): from groups that are ranked in place to
# those that send the order back to all bits (over 32 records on a side).
@pytest.mark.parametrize("m", [2, 8, 31, 32, 33, 34, 64, 65, 66, 200])
@pytest.mark.parametrize("n", [5000, 70_001])
def test_time_ordering_groups(n, m):
    rng = np.random.default_rng(n + m)
    upper = (np.arange(n) // m).astype(np.uint64) << np.uint64(34)
    low = rng.integers(0, 2 * m, n).astype(np.uint64)
    y = (np.float64(1.0).view(np.uint64) + upper + low).view(np.float64)
    rng.shuffle(y)
    status = rng.integers(0, 3, n).astype(np.int8)
    prob = ss.Problem("fg", y, status, np.array([0, n]), np.arange(n, dtype=np.int32))
    order = np.argsort(-y, kind="stable")
    np.testing.assert_array_equal(prob.perm.cpu().numpy(), order)
    inv = np.empty_like(order)
    inv[order] = np.arange(n)
    np.testing.assert_array_equal(prob.inv_perm.cpu().numpy(), inv)
    ys, st = y[order], status[order]
    end = np.append(ys[1:] != ys[:-1], True)
    run = np.concatenate([[0], np.cumsum(end)[:-1]])
    d = np.bincount(run, st == 1)
    np.testing.assert_array_equal(prob.d32.cpu().numpy(), np.where(end, d[run], 0).astype(np.int64))
    assert float(prob.c[0]) == float(np.sum(st == 1))


@pytest.mark.parametrize("n,m", [(1, 2), (700, 701), (2_100_000, 2_100_001), (3, 2**31 - 1)])
def test_design_more_entries_than_subjects(n, m):
    """A column with more entries than there are subjects has a duplicate row,
    whatever their number: refused, at the largest number of entries too."""
    if torch.cuda.mem_get_info()[0] < 24 * m + 2**30:
        pytest.skip("needs %.0f GB" % (24e-9 * m))
    rows = torch.arange(m, dtype=torch.int32, device=DEV).remainder_(n)
    with pytest.raises(ss.SurvScanError):
        ss.Problem("cox", np.arange(n, dtype=np.float64), np.ones(n, dtype=np.int8),
                   np.array([0, m], dtype=np.int64), rows)
    # the device is as it was
    y = np.random.default_rng(n).random(500)
    prob = ss.Problem("cox", y, np.ones(500, dtype=np.int8), np.array([0, 1]),
                      np.array([7], dtype=np.int32))
    np.testing.assert_array_equal(prob.perm.cpu().numpy(), np.argsort(-y, kind="stable"))


def test_prepare_from_several_threads():
    """Designs of one window each, of different sizes (so different amounts of
    LDS for the same kernel), prepared by several threads on streams of
    their own."""
    import threading
    sizes = [140_000, 300_000, 600_000, 1_048_576]
    cases = []
    for n in sizes:
        rng = np.random.default_rng(n)
        rows = [np.sort(rng.choice(n, n // 50, replace=False)) for _ in range(3)]
        ptr = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
        y = rng.random(n)
        cases.append((n, y, rng.integers(0, 2, n).astype(np.int8), ptr,
                      np.concatenate(rows).astype(np.int32)))
    failed = []

    def work(c):
        try:
            n, y, st, ptr, rows = c
            order = np.argsort(-y, kind="stable")
            inv = np.empty_like(order)
            inv[order] = np.arange(n)
            want = np.concatenate([np.sort(inv[rows[a:b]]) for a, b in zip(ptr[:-1], ptr[1:])])
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(6):
                    prob = ss.Problem("cox", y, st, ptr, rows, None, DEV)
                    got = prob.rows_sorted.cpu().numpy()
                    assert np.array_equal(got, want)
        except BaseException as e:  # noqa: BLE001
            failed.append(e)

    threads = [threading.Thread(target=work, args=(c,)) for c in cases]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
