"""The products with A over the shapes at which their kernels can go wrong: rows that start on any element, a last
16-byte chunk that is only partly there, the edges of each variant's width, row counts around a workgroup's share.

Evaluations are compared with the same sums in numpy in 64 bits, iterations with the two-pass organisation, which
shares no kernel with the single read.  Bound: a sum of k products in 64 bits is off by at most k 2^-53 times the sum of
their magnitudes; with k <= 3e4 terms of like size that is below 1e-12 of the vectors' norms, and three iterations
amplify it by no more than the factors seen for well-conditioned Gaussian matrices (1e-10 is asked)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2203_16340_amd as L
import workloads
from gpu_helpers import DEV, rel_err, to_dev

pytestmark = pytest.mark.gpu

LSQ, L1, LOGI = L.OBJ_LSQ, L.OBJ_LSQ_L1SPLIT, L.OBJ_LOGISTIC_L2


def _problem(kind, rows, cols, dtype, seed, pad=0, shift=0):
    """Device matrix whose rows start `shift` elements into an allocation of leading dimension cols + pad."""
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((rows, cols)).astype(dtype)
    flat = torch.full((shift + rows * (cols + pad),), float("nan"), dtype=torch.from_numpy(A).dtype, device=DEV)
    A_d = flat[shift:].view(rows, cols + pad)[:, :cols]
    A_d.copy_(torch.from_numpy(A))
    n = 2 * cols if kind == L1 else cols
    if kind == LOGI:
        b = np.where(A @ rng.standard_normal(cols).astype(dtype) + rng.standard_normal(rows) >= 0, 1.0, -1.0)
        l, u = np.full(n, -0.5), np.full(n, 0.5)
    else:
        b = A.astype(np.float64) @ (rng.random(cols) * (rng.random(cols) < 0.3)) + 0.1 * rng.standard_normal(rows)
        l, u = np.zeros(n), np.full(n, np.inf)
    x = np.clip(rng.random(n) * 0.4, l, u)
    return A, A_d, b, l, u, x


def _solver(kind, A_d, b, l, u, m=5, extra=None, **opts):
    return L.Solver(kind, A_d, to_dev(b), to_dev(l), to_dev(u), m, lam=0.3 if kind == L1 else 0.0,
                    mu=1e-3 if kind == LOGI else 0.0, extra=extra, options=L.default_options(tol=0.0, refresh_every=0, **opts))


def _reference_fg(kind, A, b, x):
    A = A.astype(np.float64)
    c = A.shape[1]
    if kind == LOGI:
        z = A @ x
        f = np.logaddexp(0.0, -b * z).mean() + 0.5e-3 * x @ x
        return f, A.T @ (-b / (1.0 + np.exp(b * z))) / len(b) + 1e-3 * x, z
    r = A @ (x[:c] - x[c:] if kind == L1 else x) - b
    w = A.T @ r
    if kind == L1:
        return 0.5 * r @ r + 0.3 * x.sum(), np.concatenate([w + 0.3, -w + 0.3]), r
    return 0.5 * r @ r, w, r


def _check(kind, rows, cols, dtype, pad, shift):
    A, A_d, b, l, u, x = _problem(kind, rows, cols, dtype, seed=rows * 31 + cols, pad=pad, shift=shift)
    print(f"kind {kind} rows {rows} cols {cols} {np.dtype(dtype).name} pad {pad} shift {shift}", flush=True)
    s = _solver(kind, A_d, b, l, u)
    assert s.apass_name == "fused"
    f, g, row = s.dbg_fg(to_dev(x), want_rowvec=True)
    f_ref, g_ref, row_ref = _reference_fg(kind, A, b, x)
    assert abs(f - f_ref) <= 1e-12 * abs(f_ref)
    assert rel_err(g.cpu().numpy(), g_ref) <= 1e-12
    assert rel_err(row.cpu().numpy(), row_ref) <= 1e-12
    two = _solver(kind, A_d, b, l, u, a_pass=L.APASS_TWO_PASS)
    for sol in (s, two):
        sol.set_x(to_dev(x))
    for _ in range(3):
        s.step(False)
        two.step(False)
    if cols >= 16:                        # (fewer variables may be at the solution, or at a bound, after one iteration)
        assert s.info().iters == two.info().iters == 3
        assert rel_err(s.g().cpu().numpy(), two.g().cpu().numpy()) <= 1e-10
    assert rel_err(s.x().cpu().numpy(), two.x().cpu().numpy()) <= 1e-10


# one shape around every variant's upper width, with every remainder of a chunk among them
RAGGED = [(LSQ, np.float64, c) for c in (301, 1023, 1025, 2047, 5121, 10239, 20427, 20429, 22529)]
RAGGED += [(LSQ, np.float32, c) for c in (301, 510, 513, 1023, 1025, 2050, 5119, 10242, 20425)]
RAGGED += [(LOGI, np.float64, c) for c in (301, 1025, 2049, 5119, 10241)]
RAGGED += [(LOGI, np.float32, c) for c in (301, 511, 1025, 2049, 5121, 10243)]
RAGGED += [(L1, np.float64, 1025), (L1, np.float32, 2051)]


@pytest.mark.parametrize("kind,dtype,cols", RAGGED)
def test_rows_on_any_element(kind, dtype, cols):
    _check(kind, 517, cols, dtype, pad=0, shift=1)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("pad,shift", [(0, 0), (1, 0), (3, 3), (4, 2)])
def test_leading_dimension_and_start(dtype, pad, shift):
    """Whole chunks on unaligned rows, and the elements between the rows (NaN here) are not touched."""
    _check(LSQ, 300, 1200, dtype, pad, shift)
    _check(LOGI, 300, 1200, dtype, pad, shift)


def test_unaligned_rows_asked_for_by_name_are_refused():
    _, A_d, b, l, u, _ = _problem(LSQ, 300, 1201, np.float64, seed=1)
    with pytest.raises(L.LbfgsbError) as e:
        _solver(LSQ, A_d, b, l, u, a_pass=L.APASS_FUSED)
    assert e.value.code == L.E_UNSUPPORTED


def _backtracking(rows, cols, dtype, seed, first=True):
    """Badly scaled features: the first step is halved a dozen times and more; first = False: steps in between, once or
    twice.  Returns the problem and the oracle's rejected trial steps of the first six iterations."""
    how = dict(feature_scale=20, column_spread=2, bound=5.0, label_noise=0.5, mu=1e-3) if first else \
        dict(feature_scale=1, column_spread=1.5, bound=50.0, random_start=True, label_noise=0.0, mu=1e-6)
    prob = workloads.logistic(rows=rows, cols=cols, seed=seed, dtype=np.float64, m=5, **how)
    prob.A = np.ascontiguousarray(prob.A.astype(dtype))
    orc = oracle.Solver(oracle.Objective(prob.kind, prob.A, prob.b, prob.lam, prob.mu), prob.l, prob.u, prob.x0, prob.m,
                        oracle.default_options(tol=0.0))
    counts = []
    for _ in range(6):
        orc.step()
        counts.append(orc.info.backtracks)
    orc.close()
    return prob, counts


@pytest.mark.parametrize("dtype,rows,cols,first", [(np.float32, 900, 403, False), (np.float32, 900, 403, True),
                                                   (np.float64, 517, 1025, True), (np.float64, 600, 20426, True)])
def test_logistic_steps_that_finish_on_the_device_replayed_from_a_graph(dtype, rows, cols, first):
    """Steps recorded on unaligned rows, and on rows so wide that the numbers per row of the short launch sequence do not
    fit LDS beside v (20426 columns: 16 bytes are left of it, a workgroup has 3 rows), finish every iteration on the device,
    also one whose first trial step is rejected: x is right although the host does not look in between.  (The look at x
    before the first replay is the last that the library takes: it knows of no steps after it.)"""
    prob, counts = _backtracking(rows, cols, dtype, seed=0, first=first)
    assert max(counts[:5]) >= 1
    eager = L.solver_for_problem(prob, DEV, tol=0.0, a_pass=L.APASS_AUTO)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        rec = L.solver_for_problem(prob, DEV, tol=0.0, a_pass=L.APASS_AUTO)
        assert rec.apass_name == "fused"
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            rec.step(False)
        rec.x()
    torch.cuda.synchronize()
    for _ in range(5):
        graph.replay()
        torch.cuda.synchronize()
        eager.step(False)
        assert rel_err(rec.x().cpu().numpy(), eager.x().cpu().numpy()) <= 1e-12
    assert max(r.backtracks for r in eager.history()) >= 1


# a ragged width of every logistic variant of the kernel for narrow rows, and of the ring kernel's; rows past the first
# tile of every wave (512 workgroups of four) for the variants that hold four sets of rows
REJECTED = [(np.float32, 517, c) for c in (31, 63, 95, 127, 191, 255, 383, 511, 767, 1537, 2049, 5121, 10243)]
REJECTED += [(np.float64, 517, c) for c in (15, 31, 47, 63, 95, 127, 191, 255, 383, 769, 1025, 2049, 5119, 10241)]
REJECTED += [(np.float32, 8201, c) for c in (1023, 1279, 1535)] + [(np.float64, 8201, c) for c in (511, 639, 767)]


@pytest.mark.parametrize("dtype,rows,cols", REJECTED)
def test_columns_after_a_rejected_first_trial_step(dtype, rows, cols):
    """The step that is accepted in the end is not the one whose columns the single read has formed: they are formed anew,
    by the kernel of the shape or the transposed pass.  Against the two-pass kernels over the first iterations, with and
    without a look after every step."""
    prob, counts = _backtracking(rows, cols, dtype, seed=cols)
    assert counts[0] >= 1
    print(f"rows {rows} cols {cols} {np.dtype(dtype).name} rejected {counts}", flush=True)
    s, ahead, two = (L.solver_for_problem(prob, DEV, tol=0.0, a_pass=p) for p in (L.APASS_AUTO, L.APASS_AUTO, L.APASS_TWO_PASS))
    assert s.apass_name == "fused"
    for k in range(3):
        a, b = s.step(), two.step()
        ahead.step(False)
        assert (a.status, a.iters, a.branch, a.backtracks, a.n_fixed) == (b.status, b.iters, b.branch, b.backtracks, b.n_fixed)
        assert a.backtracks == counts[k]
        assert rel_err(s.g().cpu().numpy(), two.g().cpu().numpy()) <= 1e-9
    assert rel_err(s.x().cpu().numpy(), two.x().cpu().numpy()) <= 1e-10
    assert torch.equal(ahead.x(), s.x()) and torch.equal(ahead.g(), s.g())


def test_static_solve_of_unaligned_rows_that_fit_only_without_the_single_read():
    """The single-read pass would need 40 MB of partial columns: the call still runs, on the two-pass kernels."""
    A, A_d, b, l, u, x = _problem(LSQ, 900, 20001, np.float32, seed=6)
    opts = L.default_options(tol=0.0, max_iter=3)
    ref = L.Solver(LSQ, A_d, to_dev(b), to_dev(l), to_dev(u), 5, options=opts)
    assert ref.workspace.numel() > L.STATIC_SCRATCH_BYTES
    ref.set_x(to_dev(x))
    ref.solve()
    x_d = to_dev(x)
    info = L.solve_static(LSQ, A_d, to_dev(b), to_dev(l), to_dev(u), 5, x_d, options=opts)
    assert info.iters == 3
    assert rel_err(x_d.cpu().numpy(), ref.x().cpu().numpy()) <= 1e-10


def test_static_solve_of_unaligned_narrow_rows_that_fit_only_without_the_single_read():
    """The pass for narrow rows would need 6 MB of partial columns beside 27 MB of row vectors."""
    rows, cols = 1_140_000, 1535
    gen = torch.Generator(device=DEV)
    gen.manual_seed(6)
    A_d = torch.randn(rows, cols, dtype=torch.float32, device=DEV, generator=gen)
    b_d = 10.0 * torch.randn(rows, dtype=torch.float64, device=DEV, generator=gen) + A_d[:, 0].double()
    l, u = np.zeros(cols), np.full(cols, np.inf)
    x = np.random.default_rng(6).random(cols) * 0.4
    opts = L.default_options(tol=0.0, max_iter=3)
    ref = L.Solver(LSQ, A_d, b_d, to_dev(l), to_dev(u), 5, options=opts)
    assert ref.workspace.numel() > L.STATIC_SCRATCH_BYTES
    ref.set_x(to_dev(x))
    ref.solve()
    x_d = to_dev(x)
    info = L.solve_static(LSQ, A_d, b_d, to_dev(l), to_dev(u), 5, x_d, options=opts)
    assert info.iters == 3
    assert rel_err(x_d.cpu().numpy(), ref.x().cpu().numpy()) <= 1e-10


# the kernel for narrow rows: both sides of every variant's capacity (16-byte chunks 8, 16, 24, 32, 48, 64, 96, 128, 192,
# 256), ragged widths among them, and row counts around a set (8 rows) and a tile (64 rows)
NARROW = [4 * c + d for c in (8, 16, 24, 32, 48, 64, 96, 128, 192) for d in (-1, 0, 1)] + [4, 5, 1023, 1024]


@pytest.mark.parametrize("kind", [LSQ, LOGI, L1])
@pytest.mark.parametrize("cols", NARROW)
def test_narrow_rows_fp32(kind, cols):
    _check(kind, 1203, cols, np.float32, pad=0, shift=0)


@pytest.mark.parametrize("kind", [LSQ, LOGI, L1])
@pytest.mark.parametrize("cols", [c // 2 for c in NARROW] + [5, 511])
def test_narrow_rows_fp64(kind, cols):
    _check(kind, 1203, cols, np.float64, pad=0, shift=0)


@pytest.mark.parametrize("kind", [L1, LOGI])
@pytest.mark.parametrize("rows", [8, 9, 15, 63, 64, 65, 511, 16385, 131077])
def test_narrow_row_counts(kind, rows):
    _check(kind, rows, 6, np.float32, pad=1, shift=0)
    if rows < 20000:
        _check(kind, rows, 300, np.float64, pad=0, shift=0)


# the variants that hold four sets of rows: both sides of the widest one's capacity, and rows past the first tile of every
# wave (four rows each in 512 workgroups of four), in part and in whole
@pytest.mark.parametrize("kind", [LSQ, LOGI])
@pytest.mark.parametrize("dtype,cols", [(np.float32, c) for c in (1281, 1535, 1536, 1537)] + [(np.float64, c) for c in (641, 767, 768, 769)])
def test_narrow_rows_at_the_widest(kind, dtype, cols):
    _check(kind, 1203, cols, dtype, pad=0, shift=0)


@pytest.mark.parametrize("rows", [8193, 16387])
@pytest.mark.parametrize("kind,dtype,cols", [(LOGI, np.float32, 1023), (LOGI, np.float32, 1279), (LSQ, np.float32, 1279),
                                             (LOGI, np.float32, 1535), (LSQ, np.float32, 1535), (LOGI, np.float64, 511),
                                             (LOGI, np.float64, 639), (LSQ, np.float64, 639), (LOGI, np.float64, 767),
                                             (LSQ, np.float64, 767), (LSQ, np.float64, 1023)])
def test_narrow_rows_past_the_first_tile(kind, dtype, cols, rows):
    _check(kind, rows, cols, dtype, pad=0, shift=0)


def test_narrow_row_weights():
    """Weighted least squares on narrow rows: f, g and the residual against numpy."""
    A, A_d, b, l, u, x = _problem(LSQ, 1000, 75, np.float64, seed=8)
    w = np.random.default_rng(9).random(1000) + 0.1
    s = L.Solver(LSQ, A_d, to_dev(b), to_dev(l), to_dev(u), 5, row_weight=to_dev(w), options=L.default_options(a_pass=L.APASS_AUTO))
    assert s.apass_name == "fused"
    f, g, row = s.dbg_fg(to_dev(x), want_rowvec=True)
    r = A @ x - b
    assert abs(f - 0.5 * (w * r) @ r) <= 1e-12 * f
    assert rel_err(g.cpu().numpy(), A.T @ (w * r)) <= 1e-12 and rel_err(row.cpu().numpy(), r) <= 1e-12


# vectors too long for the kernel that does the direction's work in one workgroup (more than 20 pairs: any), narrow rows of
# 32 or 64 lanes: the pass makes Algorithm 2's choice itself from the direction kernel's partial sums, with even n and up to
# 10 pairs on a copy of the scalar block that its first wave moves into place
CHOICE = [(kind, np.float32, c, 21) for c in (255, 383, 511, 767, 1023, 1279, 1535) for kind in (LSQ, LOGI)]
CHOICE += [(kind, np.float64, c, 21) for c in (127, 191, 255, 383, 511, 639, 767) for kind in (LSQ, LOGI)] + [(LSQ, np.float64, 1023, 21)]
CHOICE += [(L1, np.float64, 600, 10), (L1, np.float32, 767, 9), (LSQ, np.float32, 1100, 10), (LOGI, np.float32, 1536, 10), (LOGI, np.float32, 1535, 10)]


def _compare_steps(s, two, x, steps):
    for sol in (s, two):
        sol.set_x(to_dev(x))
    for _ in range(steps):
        a, b = s.step(), two.step()
        assert (a.status, a.iters, a.branch, a.backtracks, a.n_fixed, a.pairs_used) == \
            (b.status, b.iters, b.branch, b.backtracks, b.n_fixed, b.pairs_used)
        assert a.gp == pytest.approx(b.gp, rel=1e-9) and a.alpha_ub == pytest.approx(b.alpha_ub, rel=1e-9)
    assert rel_err(s.x().cpu().numpy(), two.x().cpu().numpy()) <= 1e-10
    assert rel_err(s.g().cpu().numpy(), two.g().cpu().numpy()) <= 1e-10


@pytest.mark.parametrize("kind,dtype,cols,m", CHOICE)
def test_narrow_pass_that_makes_the_choice(kind, dtype, cols, m):
    A, A_d, b, l, u, x = _problem(kind, 2000, cols, dtype, seed=cols + m)
    print(f"kind {kind} cols {cols} {np.dtype(dtype).name} m {m}", flush=True)
    s, two = (_solver(kind, A_d, b, l, u, m=m, a_pass=p) for p in (L.APASS_AUTO, L.APASS_TWO_PASS))
    _compare_steps(s, two, x, 5)


@pytest.mark.parametrize("n_extra", [1, 2, 3])
@pytest.mark.parametrize("cols,m", [(600, 21), (1500, 10)])
def test_narrow_pass_that_makes_the_choice_with_extra_rows(n_extra, cols, m):
    """One or two extra rows ride along with the direction kernel, three have a kernel that reads the choice."""
    A, A_d, b, l, u, x = _problem(LSQ, 2500, cols, np.float32, seed=cols + n_extra)
    rng = np.random.default_rng(cols)
    extra = (to_dev(rng.standard_normal((n_extra, cols))), to_dev(rng.standard_normal(n_extra)), to_dev(rng.random(n_extra) + 5.0))
    s, two = (_solver(LSQ, A_d, b, l, u, m=m, extra=extra, a_pass=p) for p in (L.APASS_AUTO, L.APASS_TWO_PASS))
    _compare_steps(s, two, x, 5)


# the quadratic form's products from the upper triangle (from 4096 variables on): one strip of 512 columns more or less,
# ragged last strips and chunks, unaligned rows; a size on either side that belongs to the row kernels
@pytest.mark.parametrize("n", [4095, 4096, 4097, 4607, 4608, 4609, 5121, 15872, 15873])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("signed", [False, True])
def test_symmetric_products(n, dtype, signed):
    if n > 15000 and signed:
        pytest.skip("the widest matrices once only")
    rng = np.random.default_rng(n)
    B = rng.standard_normal((n, n), dtype=dtype)
    K = (B + B.T) / 2
    K[np.diag_indices(n)] += dtype(2.0 * np.sqrt(n))
    K64 = K.astype(np.float64)
    q, x = rng.standard_normal(n), rng.random(n)
    sign = np.where(rng.random(n) < 0.5, -1.0, 1.0) if signed else np.ones(n)
    l, u = np.zeros(n), np.full(n, 1.0)

    def solver(**opts):
        return L.Solver(L.OBJ_QP, torch.from_numpy(K).to(DEV), to_dev(q), to_dev(l), to_dev(u), 5,
                        sign=to_dev(sign) if signed else None, options=L.default_options(tol=0.0, refresh_every=0, **opts))

    print(f"n {n} {np.dtype(dtype).name} signed {signed}", flush=True)
    s, two = solver(), solver(a_pass=L.APASS_TWO_PASS)
    f, g, row = s.dbg_fg(to_dev(x), want_rowvec=True)
    v = sign * x
    t = K64 @ v
    assert rel_err(row.cpu().numpy(), t) <= 1e-12
    assert rel_err(g.cpu().numpy(), sign * t + q) <= 1e-12
    assert abs(f - (0.5 * v @ t + q @ x)) <= 1e-12 * np.linalg.norm(v) * np.linalg.norm(t)
    for sol in (s, two):
        sol.set_x(to_dev(x))
    for _ in range(3):
        a, b = s.step(), two.step()
        assert (a.status, a.branch, a.backtracks, a.n_fixed) == (b.status, b.branch, b.backtracks, b.n_fixed)
        assert a.f == pytest.approx(b.f, rel=1e-10)
    assert rel_err(s.x().cpu().numpy(), two.x().cpu().numpy()) <= 1e-10
    assert rel_err(s.g().cpu().numpy(), two.g().cpu().numpy()) <= 1e-10


def test_symmetric_products_lose_no_precision():
    """The products from the upper triangle are sums of row halves and column halves: no further from the exact ones than
    the two-pass kernel's, which adds whole rows.  (Measured: 0.68 and 0.76 times 2^-53; with one chain of additions per
    column of a wave it was 1.08.  Four vectors of one sign and 400 rows each: the figures vary by 3 %.)"""
    n = 4608
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 20)) / np.sqrt(20.0)
    sq = (X * X).sum(1)
    K = np.exp(-np.maximum(sq[:, None] + sq[None, :] - 2.0 * (X @ X.T), 0.0))
    K = 0.5 * (K + K.T)
    l, u = to_dev(np.zeros(n)), to_dev(np.ones(n))
    error = {}
    for a_pass in (L.APASS_AUTO, L.APASS_TWO_PASS):
        s = L.Solver(L.OBJ_QP, to_dev(K), to_dev(-np.ones(n)), l, u, 5, options=L.default_options(a_pass=a_pass))
        rng = np.random.default_rng(1)
        total = 0.0
        for _ in range(4):
            v, rows = rng.random(n), rng.choice(n, 400, replace=False)
            _, _, t = s.dbg_fg(to_dev(v), want_rowvec=True)
            exact = (K[rows].astype(np.longdouble) * v).sum(1)
            total += float(np.linalg.norm(t.cpu().numpy()[rows] - exact) / np.linalg.norm(exact)) ** 2
        error[a_pass] = np.sqrt(total / 4) * 2.0 ** 53
        s.close()
    print(error, flush=True)
    assert error[L.APASS_AUTO] <= error[L.APASS_TWO_PASS]


@pytest.mark.parametrize("cols,bound", [(1500, 1.75), (1100, 1.65)])
def test_narrow_row_sums_lose_no_precision(cols, bound):
    """Residuals of Gaussian fp32 rows against 80-bit sums.  (Measured over eight draws in units of 2^-53: 1.61 and 1.55, the
    ring kernel 1.63 and 1.59; with one chain of additions per lane 1.90 and 1.75.  400 rows of four draws each: the figures
    vary by 2 %.)"""
    total = 0.0
    for seed in range(4):
        rng = np.random.default_rng(seed)
        A = rng.standard_normal((2500, cols)).astype(np.float32)
        b, x, rows = -rng.random(2500), rng.random(cols), rng.choice(2500, 400, replace=False)
        s = _solver(LSQ, to_dev(A), b, np.zeros(cols), np.full(cols, np.inf))
        _, _, r = s.dbg_fg(to_dev(x), want_rowvec=True)
        exact = (A[rows].astype(np.longdouble) * x).sum(1) - b[rows]
        total += float(np.linalg.norm(r.cpu().numpy()[rows] - exact) / np.linalg.norm(exact)) ** 2
        s.close()
    error = np.sqrt(total / 4) * 2.0 ** 53
    print(error, flush=True)
    assert error <= bound


@pytest.mark.parametrize("n,dtype,pad,name", [(301, np.float64, 0, "two_pass"), (1024, np.float64, 1, "two_pass"), (1025, np.float64, 0, "two_pass"),
                                              (4095, np.float64, 0, "two_pass"), (4097, np.float64, 0, "fused"),
                                              (1023, np.float32, 0, "two_pass"), (2599, np.float32, 0, "two_pass"),
                                              (2601, np.float32, 0, "fused"), (4096, np.float32, 1, "fused"),
                                              (1024, np.float64, 0, "fused"), (2500, np.float32, 0, "fused")])
def test_row_products_of_the_quadratic_form(n, dtype, pad, name):
    """One product with the matrix in either organisation: on rows that start on any element four rows per wave (k_gemv)
    where that is the faster kernel (up to 15 % of an iteration), as before the ring kernel took such rows."""
    rng = np.random.default_rng(n)
    B = rng.standard_normal((n, n)).astype(dtype)
    K = (B + B.T) / 2 + np.diag(np.full(n, 2.0 * np.sqrt(n), dtype))
    K_d = torch.full((n, n + pad), float("nan"), dtype=torch.from_numpy(K).dtype, device=DEV)[:, :n]
    K_d.copy_(torch.from_numpy(K))
    q, x = rng.standard_normal(n), rng.random(n)
    s = L.Solver(L.OBJ_QP, K_d, to_dev(q), to_dev(np.zeros(n)), to_dev(np.ones(n)), 5, options=L.default_options(tol=0.0))
    assert s.apass_name == name
    f, g, row = s.dbg_fg(to_dev(x), want_rowvec=True)
    t = K.astype(np.float64) @ x
    assert rel_err(row.cpu().numpy(), t) <= 1e-12 and rel_err(g.cpu().numpy(), t + q) <= 1e-12
    assert abs(f - (0.5 * x @ t + q @ x)) <= 1e-12 * np.linalg.norm(x) * np.linalg.norm(t)
    s.close()
