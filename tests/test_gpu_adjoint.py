"""GPU: the full gradient in eta (ss_eta_gradient) against the oracle.

Checks, element by element on the same seeded inputs:
  * dl/deta against oracle.adjoint.eta_gradient_scan (itself pinned to the
    chain-rule definition and to complex steps on the CPU), each element
    within 1e-10 of its condition scale delta_m + e_m * (inner sum);
  * l against oracle.adjoint.loglik_eta, within 1e-10 of
    sum |delta eta| + sum d |log S0|;
  * x_j' (dl/deta) = g' of coordinate j from ss_grad_hess (both GPU paths,
    property that holds at any size) -- the link the proximal-gradient step
    of Sec. 2.9 relies on;
  * the autograd wrapper: backward equals the gradient, and torch's
    finite-difference gradcheck passes on a small case.
Edge cases: one subject, all censored (gradient zero, l = 0), all events,
heavy ties, a ragged size across many scan tiles, the N = 1e6 sweep design.
"""
import numpy as np
import pytest

from oracle import adjoint as oadj, prep as oprep, scan as oscan

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2204_08183_amd import survscan as ss  # noqa: E402

from test_gpu_parity import make_case, gpu_problem, xcol  # noqa: E402

DEV = "cuda:0"
TOL = 1e-10


def check_gradient(model, c, prob=None):
    prob = prob or gpu_problem(model, c)
    grad, ll = prob.eta_gradient()
    got = grad.cpu().numpy()
    want = oadj.eta_gradient_scan(model, c["y"], c["status"], c["eta"])
    ev = oprep.event_indicator(model, c["status"]).astype(np.float64)
    scale = ev + np.abs(ev - want)            # delta_m + e_m * inner_m
    err = np.abs(got - want) / np.maximum(scale, 1e-300)
    assert float(err.max(initial=0.0)) <= TOL, (model, c["n"], float(err.max()),
                                                int(err.argmax()))
    want_l = oadj.loglik_eta(model, c["y"], c["status"], c["eta"])
    l_scale = float(np.sum(np.abs(c["eta"] * ev))) + abs(want_l) + 1.0
    assert abs(float(ll.cpu()[0]) - want_l) <= TOL * l_scale, (float(ll.cpu()[0]), want_l)
    return prob, got


CASES = [("cox", 1000, 3, 0, 0, False), ("cox", 50001, 4, 1, 40, False),
         ("cox", 20000, 3, 2, 0, True), ("fg", 1000, 3, 3, 0, False),
         ("fg", 50001, 4, 4, 40, False), ("fg", 20000, 3, 5, 0, True)]


@pytest.mark.parametrize("model,n,p,seed,ties,valued", CASES)
def test_eta_gradient_matches_oracle(model, n, p, seed, ties, valued):
    c = make_case(model, n, p, seed, ties, 0.1, valued)
    prob, got = check_gradient(model, c)
    # x_j' grad = g' (GPU fused coordinate kernel) for every column
    for j in range(p):
        x = xcol(c, j)
        g1 = float(prob.grad_hess(j).cpu()[0])
        scale = float(np.sum(np.abs(x) * (np.abs(got) + 1.0)))
        assert abs(float(x @ got) - g1) <= TOL * scale, (model, j, float(x @ got), g1)


@pytest.mark.parametrize("model", ["cox", "fg"])
def test_eta_gradient_edges(model):
    # one subject
    c = make_case(model, 1, 1, 6, 0, 1.0, False)
    check_gradient(model, c)
    # everything censored: no events, gradient zero, l = 0
    c = make_case(model, 3000, 2, 7, 0, 0.2, False, status="censored")
    prob, got = check_gradient(model, c)
    assert np.all(got == 0.0)
    assert float(prob.eta_gradient()[1].cpu()[0]) == 0.0
    # every subject an event of interest
    c = make_case(model, 3000, 2, 8, 5, 0.2, False, status="events")
    check_gradient(model, c)
    # one tie run holding every subject
    c = make_case(model, 2049, 2, 9, 0, 0.2, False)
    c["y"] = np.full(c["n"], 1.5)
    check_gradient(model, c)
    # ragged size across many scan tiles, large eta offset
    c = make_case(model, 262145, 2, 10, 0, 0.05, False, eta_shift=30.0)
    check_gradient(model, c)


def test_eta_gradient_sweep_design():
    """The N = 1e6, P = 1000 design of the l1 CCD sweep (one column set per
    model), at the eta a partial sweep leaves."""
    import gen
    for model in ("cox", "fg"):
        d = gen.cox_data(0, 1_000_000, 50, 0.05) if model == "cox" else \
            gen.fg_data(0, 1_000_000, 50, 0.05)
        rng = np.random.default_rng(12)
        c = {"y": d["y"], "status": d["status"], "col_ptr": d["col_ptr"], "rows": d["rows"],
             "vals": None, "eta": rng.normal(0.0, 0.5, d["n"]), "n": d["n"], "p": d["p"]}
        prob, got = check_gradient(model, c)
        pr = oscan.Prepared(model, c["y"], c["status"])
        for j in (0, 17, 49):
            x = xcol(c, j)
            want = pr.coordinate(c["eta"], x)
            assert abs(float(x @ got) - want["g1"]) <= TOL * want["scale_g1"] * 10


def test_eta_gradient_rejects_bad_arguments():
    c = make_case("cox", 1000, 1, 11, 0, 0.2, False)
    prob = gpu_problem("cox", c)
    lib = ss.load()
    grad = torch.empty(prob.n, dtype=torch.float64, device=DEV)
    ll = torch.empty(1, dtype=torch.float64, device=DEV)
    ws = ss.Workspace(lib.ss_eta_gradient_workspace_bytes(prob.n), DEV)
    args = [prob.perm.data_ptr(), prob.status.data_ptr(), prob.eta.data_ptr(),
            prob.e.data_ptr(), prob.d8.data_ptr(), prob.d32.data_ptr(), None, None,
            grad.data_ptr(), ll.data_ptr()]
    assert lib.ss_eta_gradient(7, prob.n, *args, ws.ptr, ws.nbytes, None) == ss.SS_EUNSUPPORTED
    assert lib.ss_eta_gradient(ss.COX, 0, *args, ws.ptr, ws.nbytes, None) == ss.SS_EINVAL
    assert lib.ss_eta_gradient(ss.COX, prob.n, *args, ws.ptr, ws.nbytes - 8,
                               None) == ss.SS_EWORKSPACE
    # Fine-Gray needs the IPCW arrays
    assert lib.ss_eta_gradient(ss.FINE_GRAY, prob.n, *args, ws.ptr, ws.nbytes,
                               None) == ss.SS_EINVAL
    assert lib.ss_eta_gradient_workspace_bytes(0) == 0


@pytest.mark.parametrize("model", ["cox", "fg"])
def test_loglik_eta_autograd(model):
    c = make_case(model, 5000, 1, 13, 10, 0.2, False)
    prob = gpu_problem(model, c)
    eta = torch.tensor(c["eta"], dtype=torch.float64, device=DEV, requires_grad=True)
    l = ss.loglik_eta(prob, eta)
    (2.5 * l).backward()
    want = oadj.eta_gradient_scan(model, c["y"], c["status"], c["eta"])
    got = eta.grad.cpu().numpy()
    ev = oprep.event_indicator(model, c["status"]).astype(np.float64)
    assert np.max(np.abs(got - 2.5 * want) / (2.5 * (ev + np.abs(ev - want)))) <= TOL
    # finite differences through the GPU forward pass (small case)
    c = make_case(model, 60, 1, 14, 3, 0.2, False)
    small = gpu_problem(model, c)
    eta = torch.tensor(c["eta"], dtype=torch.float64, device=DEV, requires_grad=True)
    assert torch.autograd.gradcheck(lambda t: ss.loglik_eta(small, t), (eta,), eps=1e-6,
                                    atol=1e-7, rtol=1e-6)


# ---------------------------------------------------------------- X' (dl/deta)
BETA_CASES = CASES + [("cox", 1, 2, 40, 0, False), ("fg", 2, 2, 41, 0, True),
                      ("cox", 200_003, 6, 42, 900, True), ("fg", 131_073, 5, 43, 0, False)]


@pytest.mark.parametrize("model,n,p,seed,ties,valued", BETA_CASES)
def test_beta_gradient_matches_oracle(model, n, p, seed, ties, valued):
    """ss_beta_gradient: X' times the oracle's gradient in eta, column by
    column, within 1e-10 of sum |x| (|dl/deta| + 1); l as the oracle's;
    the optional subject-order gradient equals ss_eta_gradient's; and each
    entry equals g' of the fused coordinate kernel (a different algorithm)."""
    c = make_case(model, n, p, seed, ties, 0.1, valued)
    prob = gpu_problem(model, c)
    grad_eta = torch.empty(n, dtype=torch.float64, device=DEV)
    gb, ll = prob.beta_gradient(grad_eta=grad_eta)
    got = gb.cpu().numpy()
    want_eta = oadj.eta_gradient_scan(model, c["y"], c["status"], c["eta"])
    want_l = oadj.loglik_eta(model, c["y"], c["status"], c["eta"])
    ev = oprep.event_indicator(model, c["status"]).astype(np.float64)
    l_scale = float(np.sum(np.abs(c["eta"] * ev))) + abs(want_l) + 1.0
    assert abs(float(ll.cpu()[0]) - want_l) <= TOL * l_scale
    for j in range(p):
        x = xcol(c, j)
        scale = float(np.sum(np.abs(x) * (np.abs(want_eta) + 1.0)))
        assert abs(got[j] - float(x @ want_eta)) <= TOL * scale, (model, n, j)
        g1 = float(prob.grad_hess(j).cpu()[0])
        assert abs(got[j] - g1) <= TOL * scale, (model, n, j, got[j], g1)
    ge, _ = prob.eta_gradient()
    np.testing.assert_array_equal(grad_eta.cpu().numpy(), ge.cpu().numpy())
    # without the subject-order output the sums are the same (deterministic)
    gb2, _ = prob.beta_gradient()
    np.testing.assert_array_equal(gb2.cpu().numpy(), got)
    assert prob.workspace_error() == 0


@pytest.mark.parametrize("model", ["cox", "fg"])
def test_beta_gradient_paper_scale(model):
    """N = 1e6, P = 1000 (the Sec. 3.2 design) at the generating
    coefficients: every entry of X' (dl/deta) against g' of ss_grad_hess
    (property at any size), sampled columns against the oracle's scan."""
    import gen
    d = gen.cox_data(0, 1_000_000, 1000, 0.05) if model == "cox" else \
        gen.fg_data(0, 1_000_000, 1000, 0.05)
    eta = gen.linear_predictor(d["n"], d["col_ptr"], d["rows"], None, d["beta_true"])
    prob = ss.Problem(model, d["y"], d["status"], d["col_ptr"], d["rows"], None, DEV)
    prob.set_eta(eta)
    gb, _ = prob.beta_gradient()
    got = gb.cpu().numpy()
    g = torch.empty((1000, 3), dtype=torch.float64, device=DEV)
    for j in range(1000):
        prob.grad_hess(j, out=g[j])
    g1 = g[:, 0].cpu().numpy()
    cnt = np.diff(d["col_ptr"]).astype(np.float64)
    # |x_j' g| <= sum |x_j| (|grad| + 1) <= 2 * (number of events + nnz_j)
    scale = 2.0 * (cnt + d["n"])
    assert np.all(np.abs(got - g1) <= TOL * scale)
    pr = oscan.Prepared(model, d["y"], d["status"])
    for j in (0, 500, 999):
        x = gen.dense_column(d["n"], d["col_ptr"], d["rows"], None, j)
        want = pr.coordinate(eta, x)
        assert abs(got[j] - want["g1"]) <= TOL * want["scale_g1"], j


@pytest.mark.parametrize("model", ["cox", "fg"])
def test_beta_gradient_wide_design(model):
    """A design wider than long (N = 40000, P = 30000 sparse indicator
    columns, ties): the spans of the X' pass grow to keep the partials
    within 2 (N + P), and every entry still equals X' of the oracle's
    gradient in eta (sparse product in subject order)."""
    import scipy.sparse as sp
    n, p = 40_000, 30_000
    c = make_case(model, n, p, 44, 30, 0.0005, False)
    prob = gpu_problem(model, c)
    lib = ss.load()
    assert lib.ss_beta_gradient_workspace_bytes(n, p) <= \
        lib.ss_eta_gradient_workspace_bytes(n) + 16 * (n + p) + 256
    gb, _ = prob.beta_gradient()
    got = gb.cpu().numpy()
    want_eta = oadj.eta_gradient_scan(model, c["y"], c["status"], c["eta"])
    x = sp.csc_matrix((np.ones(c["rows"].size), c["rows"], c["col_ptr"]), shape=(n, p))
    want = x.T @ want_eta
    scale = x.T @ (np.abs(want_eta) + 1.0)
    assert np.all(np.abs(got - want) <= TOL * scale), np.max(np.abs(got - want) / scale)
    assert prob.workspace_error() == 0


# ------------------------------------------- dispatch lines of the two passes
@pytest.mark.parametrize("model", ["cox", "fg"])
@pytest.mark.parametrize("n", [2047, 2049, 4_194_304, 4_194_305])
def test_eta_gradient_tile_carries(model, n):
    """One, two, 2048 and 2049 tiles of 2048 positions: up to 2048 the
    workgroups add the tile sums themselves, above a launch scans them."""
    c = make_case(model, n, 1, 45, 0, 0.001, False)
    c["y"] = np.ceil(c["y"] * n)  # some tie runs
    check_gradient(model, c)


@pytest.mark.parametrize("model,n,p,valued", [
    ("cox", 6_250_000, 15, False), ("fg", 6_250_000, 16, False), ("cox", 6_250_011, 17, True),
    ("cox", 40_000, 2499, False), ("cox", 40_000, 2500, False), ("fg", 40_009, 2530, True)])
def test_beta_gradient_column_groups(model, n, p, valued):
    """Both sides of the line between X' from L2 and from LDS (16 columns,
    1e8 positions times columns); pieces of every length around a wave's 64
    and its 512 entries in flight, a full column, a ragged last span; sampled
    columns against the oracle's gradient."""
    counts = [0, 1, 63, 64, 65, 511, 512, 513, 3000]
    rng = np.random.default_rng(p)
    rows = []
    for j in range(p):
        m = counts[j % len(counts)] if j != p - 2 else n
        # most of a column inside one span of 8192 sorted positions
        rows.append(np.arange(n) if m == n else np.sort(
            rng.permutation(min(n, 8192))[:m] + (n - min(n, 8192)) * (j % 2)))
    col_ptr = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    rows = np.concatenate(rows).astype(np.int32)
    vals = rng.normal(size=rows.size) if valued else None
    status = (rng.random(n) < 0.5).astype(np.int8)
    if model == "fg":
        status += ((status == 1) & (rng.random(n) < 0.5)).astype(np.int8)
    c = {"y": np.arange(n, 0, -1) + 0.0, "status": status, "n": n, "p": p, "col_ptr": col_ptr,
         "rows": rows, "vals": vals, "eta": rng.normal(0.0, 0.5, n)}
    got = gpu_problem(model, c).beta_gradient()[0].cpu().numpy()
    want_eta = oadj.eta_gradient_scan(model, c["y"], c["status"], c["eta"])
    for j in sorted(set(range(20)) & set(range(p)) | {p - 2, p - 1}):
        r = rows[col_ptr[j]:col_ptr[j + 1]]
        x = 1.0 if vals is None else vals[col_ptr[j]:col_ptr[j + 1]]
        scale = float(np.sum(np.abs(x) * (np.abs(want_eta[r]) + 1.0)))
        assert abs(got[j] - float(np.sum(x * want_eta[r]))) <= TOL * scale, j


@pytest.mark.parametrize("valued", [False, True])
@pytest.mark.parametrize("model,n,p", [("cox", 40_009, 2600), ("fg", 8000, 13_001),
                                       ("cox", 40_000, 30_000)])
def test_beta_gradient_sparse_columns(model, n, p, valued):
    """Batches of 64 columns none of which has more than 0, 8, 64 or 128 entries in
    a span, and batches with one that does, the columns of one
    batch all in one span or spread over all; one span or several of them,
    of one or more stretches of 8192 positions."""
    import scipy.sparse as sp
    rng = np.random.default_rng(p)
    kinds = [(0, 1), (0, 9), (8, 9), (1, 10), (0, 65), (64, 65), (60, 66), (100, 129), (120, 140)]
    cols = []
    for j in range(p):
        lo, hi = kinds[(j // 64) % len(kinds)]
        span = min(n, 8192 if (j // 576) % 2 else n)
        m = int(rng.integers(lo, hi))
        cols.append(np.sort(rng.choice(span, m, replace=False)))
    ptr = np.concatenate([[0], np.cumsum([r.size for r in cols])]).astype(np.int64)
    rows = np.concatenate(cols).astype(np.int32)
    c = make_case(model, n, 1, 46, 0, 0.001, False)
    c["y"] = -np.sort(-c["y"])  # sorted positions are the subjects
    vals = rng.normal(0.0, 1.0, rows.size) if valued else None
    prob = ss.Problem(model, c["y"], c["status"], ptr, rows, vals, DEV)
    prob.set_eta(c["eta"])
    gb, _ = prob.beta_gradient()
    want_eta = oadj.eta_gradient_scan(model, c["y"], c["status"], c["eta"])
    x = sp.csc_matrix((np.ones(rows.size) if vals is None else vals, rows, ptr), shape=(n, p))
    scale = abs(x).T @ (np.abs(want_eta) + 1.0)
    assert np.all(np.abs(gb.cpu().numpy() - x.T @ want_eta) <= TOL * scale)
    gb2, _ = prob.beta_gradient()
    assert torch.equal(gb, gb2)
