"""The Gram kernel where its layout changes: pairs per instantiation (5, 10, 20, 31 slots, part of them used), four and eight
waves per workgroup (16384 elements), one and several chunks per wave, long vectors (2^17), a last chunk of any length, vectors
that start on any element; its closing step in the kernel itself (the hook) and in the direction kernel (whole iterations).

Tolerances: sums of n products of numbers of order one in a fixed tree order, against the literal recursion's: 1e-12 normwise
(the bound of the other two-loop tests).  Iterations accumulate that through the recursion: 1e-8, as in the transport tests."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2203_16340_amd as L
from gpu_helpers import DEV, make_solver, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,pairs", [(1, 1), (5, 5), (6, 6), (10, 10), (10, 4), (11, 11), (16, 16), (20, 20), (21, 21), (31, 31)])
@pytest.mark.parametrize("n", [2, 63, 65, 4095, 16384, 16385, 33000, 65537, 131071, 131073, 131136])
def test_two_loop(n, m, pairs):
    rng = np.random.default_rng(n + 101 * m + pairs)
    S = rng.normal(size=(pairs, n))
    Y = S * np.exp(rng.normal(size=n) * 0.5) + 0.3 * S.sum(axis=1, keepdims=True) / n
    Y[pairs // 2] *= -1.0 if pairs > 2 else 1.0                     # one that fails the gate
    g, mask, yn = rng.normal(size=n), (rng.random(n) < 0.7).astype(np.uint8), np.einsum("ij,ij->i", Y, Y)
    mask[64:160] = 0                                                # chunks without a free variable
    s = make_solver(L.OBJ_LSQ, np.zeros((1, n)), np.zeros(1), np.full(n, -np.inf), np.full(n, np.inf), m)
    d, used = s.dbg_two_loop(to_dev(S), to_dev(Y), to_dev(yn), to_dev(g), to_dev(mask))
    s.close()
    ref, used_ref = oracle.two_loop(S, Y, g, mask, 1e-10, ynorm2=yn)
    d = d.cpu().numpy()
    assert used == used_ref and np.all(d[mask == 0] == 0.0)
    assert rel_err(d, ref) <= 1e-12


# tiles of four vectors: the last pair count of one, two and three tiles and the next, in a memory they fill and in one they do not
@pytest.mark.parametrize("m,pairs", [(3, 3), (4, 4), (10, 3), (10, 7), (8, 8), (10, 8), (5, 0), (10, 0)])
@pytest.mark.parametrize("n", [95, 8193, 131071, 131072, 163839])
def test_two_loop_by_pairs_held(m, pairs, n):
    rng = np.random.default_rng(n + 101 * m + pairs)
    S = rng.normal(size=(pairs, n))
    Y = S * np.exp(rng.normal(size=n) * 0.5) + 0.3 * rng.normal(size=(pairs, n))
    g, mask, yn = rng.normal(size=n), (rng.random(n) < 0.4).astype(np.uint8), np.einsum("ij,ij->i", Y, Y)
    mask[0] = 1
    s = make_solver(L.OBJ_LSQ, np.zeros((1, n)), np.zeros(1), np.full(n, -np.inf), np.full(n, np.inf), m)
    d, used = s.dbg_two_loop(to_dev(S), to_dev(Y), to_dev(yn), to_dev(g), to_dev(mask))
    s.close()
    ref, used_ref = oracle.two_loop(S, Y, g, mask, 1e-10, ynorm2=yn)
    d = d.cpu().numpy()
    assert used == used_ref and np.all(d[mask == 0] == 0.0)
    assert rel_err(d, ref) <= 1e-12


def exact_two_loop_case(c, n, seed):
    """Integer pairs with <s_i, y_i> = 3 whose every alpha_i, beta_i and result is a whole number: dividing a sum by 3 is exact
    also as a product with the rounded 1/3, where a row of G divided by 3 beforehand is rounded entry by entry.
    s_i = e_i; R holds the <s_k, y_i>, k <= i; q after the first loop is w, one coordinate; gamma = 2^-20."""
    rng = np.random.default_rng(seed)
    alpha = rng.integers(1, 10, c) * rng.choice([-1, 1], c)
    R = np.triu(rng.integers(-5, 6, (c, c)), 1) + 3 * np.eye(c, dtype=int)
    beta = -np.sign(alpha) * rng.integers(0, 6, c)
    coef = alpha - beta
    E = np.array([3 * beta[i] - coef[:i] @ R[:i, i] for i in range(c)])
    rest, squares = (3 << 20) - int(R[:, -1] @ R[:, -1]) - int(E[-1]) ** 2, []      # ||y_{c-1}||^2 = 3 2^20
    while rest:
        squares.append(math.isqrt(rest))
        rest -= squares[-1] ** 2
    S, Y, w = np.zeros((c, n)), np.zeros((c, n)), np.zeros(n)
    S[np.arange(c), np.arange(c)] = 1.0
    Y[:, :c], Y[:, c], Y[-1, c + 1:c + 1 + len(squares)], w[c] = R.T, E, squares, 1 << 20
    return S, Y, w + alpha @ Y, -(w / (1 << 20) + coef @ S)


@pytest.mark.parametrize("m,pairs", [(11, 11), (20, 11), (20, 20), (21, 21), (31, 12), (31, 31)])
@pytest.mark.parametrize("seed", range(3))
def test_the_recursion_divides_sums_not_rows(m, pairs, seed):
    S, Y, g, ref = exact_two_loop_case(pairs, pairs + 9, seed)
    n = g.size
    s = make_solver(L.OBJ_LSQ, np.zeros((1, n)), np.zeros(1), np.full(n, -np.inf), np.full(n, np.inf), m)
    d, used = s.dbg_two_loop(to_dev(S), to_dev(Y), to_dev(np.einsum("ij,ij->i", Y, Y)), to_dev(g),
                             torch.ones(n, dtype=torch.uint8, device=DEV))
    s.close()
    assert used == pairs
    np.testing.assert_array_equal(d.cpu().numpy(), ref)


# 63 504 (short vectors), 131 043 and 131 769 (odd, either side of 2^17), 131 406 entries
@pytest.mark.parametrize("rows,cols", [(252, 252), (361, 363), (363, 363), (362, 362 + 1)])
@pytest.mark.parametrize("m", [3, 10, 12])
@pytest.mark.parametrize("uniform", [True, False])
def test_iterations(rows, cols, m, uniform):
    rng = np.random.default_rng(rows + cols + m)
    M, n, rho = rng.random((rows, cols)) - 0.3, rows * cols, 4.0
    u, v = rng.random(rows) + 0.1, rng.random(cols) + 0.1
    u, v = u / u.sum(), v / v.sum()
    l, ub = np.zeros(n), np.full(n, np.inf)
    if not uniform:
        ub[rng.random(n) < 0.1] = 0.5 / n
    x0 = np.where(rng.random(n) < 0.5, 0.0, 0.4 * rng.random(n) / n)
    ref = oracle.Solver(oracle.Objective(oracle.OT_GAUSS, M, lam=0.5).set_marginals(u, v, lam=np.zeros(rows + cols), rho=rho), l, ub,
                        x0, m, oracle.default_options(tol=0.0))
    s = L.Solver(L.OBJ_OT_GAUSS, to_dev(M), to_dev(np.concatenate([u, v])), to_dev(l), to_dev(ub), m, lam=0.5,
                 options=L.default_options(tol=0.0), row_weight=to_dev(np.full(rows + cols, rho)))
    s.set_x(to_dev(x0))
    for _ in range(m + 3):
        ref.step()
        s.step(False)
    info = s.info()
    assert info.iters == ref.info.iters and info.branch == ref.info.branch and info.n_fixed == ref.info.n_fixed
    assert info.pg2 == pytest.approx(ref.info.pg2, rel=1e-8) and info.pginf == pytest.approx(ref.info.pginf, rel=1e-8)
    assert rel_err(s.x().cpu().numpy(), ref.x) <= 1e-8 and rel_err(s.g().cpu().numpy(), ref.g) <= 1e-8
    ref.close()
    s.close()


def test_a_step_after_the_end_changes_nothing():
    """Long vectors: the direction kernel finds the end of the run and leaves it to the row-sum kernel to record; further steps
    find it there."""
    rows, cols = 363, 365
    rng = np.random.default_rng(5)
    M = rng.standard_normal((rows, cols))
    n = rows * cols
    s = L.Solver(L.OBJ_OT_GAUSS, to_dev(M), None, to_dev(np.zeros(n)), to_dev(np.full(n, np.inf)), 5, lam=0.5,
                 options=L.default_options(tol=1e-9, max_iter=50))
    s.set_x(torch.zeros(n, dtype=torch.float64, device=DEV))
    for _ in range(20):
        s.step(False)
    a, xa = s.info(), s.x().clone()
    for _ in range(3):
        s.step(False)
    b = s.info()
    assert a.status == L.CONVERGED and a.as_dict() == b.as_dict() and torch.equal(xa, s.x())
    s.close()


# the resident solver's Gram matrix: one, two, three and four blocks of 16 slots (m = 7 is the last with one), vectors of fewer
# elements than one wave takes, of more than the eight waves take at once, and of a length that is no multiple of 16
@pytest.mark.parametrize("m", [1, 7, 8, 10, 16, 24, 31])
@pytest.mark.parametrize("rows,cols", [(60, 9), (200, 100), (120, 129), (90, 60)])
def test_resident_iterations(rows, cols, m):
    rng = np.random.default_rng(rows + cols + m)
    A = rng.normal(size=(rows, cols)) * np.exp(0.7 * rng.normal(size=cols))
    b = A @ np.where(rng.random(cols) < 0.5, 0.0, np.abs(rng.normal(size=cols))) + 0.1 * rng.normal(size=rows)
    l, u = np.zeros(cols), np.full(cols, np.inf)
    ref = oracle.Solver(oracle.Objective(oracle.LSQ, A, b), l, u, np.zeros(cols), m, oracle.default_options(tol=0.0))
    s = make_solver(L.OBJ_LSQ, A, b, l, u, m, tol=0.0)
    if (cols, m) == (129, 31):                           # (does not fit the compute unit's memory)
        assert s.apass_name != "resident"
        s.close()
        return
    assert s.apass_name == "resident"
    s.set_x(torch.zeros(cols, dtype=torch.float64, device=DEV))
    g0 = float(np.linalg.norm(ref.g))
    for it in range(min(m + 4, 12)):
        ref.step()
        info = s.step()
        if float(np.linalg.norm(ref.g[oracle.free_mask(ref.x, ref.g, l, u, 1e-10) != 0])) <= 1e-6 * g0:
            break                                        # (close to the minimiser the gradient is rounding)
        assert info.branch == ref.info.branch and info.backtracks == ref.info.backtracks and info.pairs_used == ref.info.pairs_used, it
        assert rel_err(s.x().cpu().numpy(), ref.x) <= 1e-8 and rel_err(s.g().cpu().numpy(), ref.g) <= 1e-7, it
    ref.close()
    s.close()


@pytest.mark.parametrize("n", [1025, 1087, 16401])
def test_what_lies_past_a_vector_does_not_count(n):
    """Ring slots that hold no pair yet, infinities in them: the newest pair's ||y||^2 ends with its vector, so the pair is used and the
    step is the same bit for bit."""
    rng = np.random.default_rng(n)
    A = to_dev(rng.standard_normal((300, n)))
    b, zero = to_dev(rng.standard_normal(300)), torch.zeros(n, dtype=torch.float64, device="cuda")
    out = []
    for planted in (False, True):
        s = L.Solver(L.OBJ_LSQ, A, b, zero, torch.full_like(zero, np.inf), 4, options=L.default_options(tol=0.0))
        s.set_x(zero)
        s.step(False)
        if planted:
            x = s.x().cpu().numpy()
            j = int(np.abs(x).argmax())
            space = s.workspace[:s.workspace.numel() // 8 * 8].view(torch.float64)
            at = [k for k in (np.nonzero(space.cpu().numpy() == x[j])[0] - j) if np.array_equal(space[k:k + n].cpu().numpy(), x)]
            y = int(at[-1]) + (4 * n + 31) // 32 * 32       # (x0 = 0: the first s is x itself; four slots of s, y begins behind them)
            assert len(at) >= 2 and np.dot(space[y:y + n].cpu().numpy(), x) > 0 and not space[y + n:y + 4 * n].any()
            space[y + n:y + 4 * n] = np.inf
        info = s.step()
        assert info.pairs_used == 1
        out.append((s.x(), s.g()))
        s.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
