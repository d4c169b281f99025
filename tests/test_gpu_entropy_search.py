"""The entropy's line search where its stages meet: the first accepted step length anywhere in the sequence of halvings, with the
first length decided from the row sums' kernel or from a launch of its own, narrow and wide workgroups, limits in every stage, and
a negative curvature, for which the search must not skip lengths.

A start at l = 1e-300 with minimisers exp(-M/lambda - 1): each constant added to M takes about three more halvings.  The
decisions are the oracle's, whole numbers; alpha = 2^-k is exact."""
import numpy as np
import pytest

import oracle
import paper_2203_16340_amd as L
from gpu_helpers import rel_err, to_dev

pytestmark = pytest.mark.gpu

LAM = 0.5


def first_iteration(rows, cols, shift, rho, max_backtracks, gpu):
    rng = np.random.default_rng(rows + cols)
    M, n = shift + 0.2 * rng.random((rows, cols)), rows * cols
    low = np.full(n, 1e-300)
    u, v = np.full(rows, 1e-3 / rows), np.full(cols, 1e-3 / cols)
    opts = dict(tol=0.0, max_backtracks=max_backtracks, eps=1e-310)
    if gpu:
        s = L.Solver(L.OBJ_OT_ENTROPY, to_dev(M), to_dev(np.concatenate([u, v])), to_dev(low), to_dev(np.full(n, np.inf)), 4, lam=LAM,
                     options=L.default_options(**opts), row_weight=to_dev(np.full(rows + cols, rho)))
        s.set_x(to_dev(low))
        info = s.step()
        x = s.x().cpu().numpy()
    else:
        obj = oracle.Objective(oracle.OT_ENTROPY, M, lam=LAM).set_marginals(u, v, lam=np.zeros(rows + cols), rho=rho)
        s = oracle.Solver(obj, low, np.full(n, np.inf), low, 4, oracle.default_options(**opts))
        s.step()
        info, x = s.info, s.x.copy()
    # (the oracle counts the gradient at the accepted point as well, and reports no halvings of a search that fails)
    if gpu:
        out = info.status, info.iters, info.backtracks, info.fevals, info.alpha, x
    else:
        out = info.status, info.iters, info.backtracks if info.iters else max_backtracks + 1, info.fevals - info.iters, info.alpha, x
    s.close()
    return out


# (with rho = 2 the penalty asks for 16 halvings at least; with rho < 0 its curvature is negative)
SHAPES = [(200, 21), (5, 4200)]   # (first length by the row sums; in its own launch)
SHIFTS = [-5.0, -4.0, -3.5, -3.0, -2.6, -2.2, -1.8, -1.4, -1.0, -0.5, 0.0, 0.5, 1.0, 1.5, 2.0, 2.5, 3.0, 4.0, 5.0, 6.0, 7.0, 9.0, 10.5, 12.0, 14.0, 16.0, 17.0, 18.0]


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("rho", [2.0, 1e-9, -1e-9])
@pytest.mark.parametrize("max_backtracks", [60, 75])
def test_accepted_lengths(rows, cols, rho, max_backtracks):
    seen = set()
    for shift in SHIFTS:
        ref = first_iteration(rows, cols, shift, rho, max_backtracks, False)
        got = first_iteration(rows, cols, shift, rho, max_backtracks, True)
        assert got[:5] == ref[:5], (shift, got[:5], ref[:5])
        assert rel_err(got[5], ref[5]) <= 1e-12, shift
        seen.add(ref[2] * ref[1])
    assert len(seen) >= (12 if rho == 2.0 else 20), seen


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("max_backtracks", [0, 1, 3, 4, 8, 9, 13, 14, 15, 16, 17, 20, 21, 22])
def test_limits(rows, cols, max_backtracks):
    for shift in (0.0, 1.0, 2.0):
        ref = first_iteration(rows, cols, shift, 2.0, max_backtracks, False)
        got = first_iteration(rows, cols, shift, 2.0, max_backtracks, True)
        assert got[:4] == ref[:4], (shift, got[:5], ref[:5])


def test_wide_workgroups():
    for shift in (0.0, 3.0, 9.0):
        ref = first_iteration(1000, 790, shift, 2.0, 60, False)
        got = first_iteration(1000, 790, shift, 2.0, 60, True)
        assert got[:5] == ref[:5], (shift, got[:5], ref[:5])
        assert rel_err(got[5], ref[5]) <= 1e-12


@pytest.mark.parametrize("rows,cols", [(1000, 790), (100, 8000)])   # (first length by the row sums; in its own launch)
@pytest.mark.parametrize("rho", [1e-9, -1e-9])
def test_first_lengths_of_wide_workgroups(rows, cols, rho):
    """The second, third and fourth length are decided without an arrival, while half of the 512 workgroups are still to begin; with a
    negative curvature all lengths are summed, 13 at a time, and decided behind one."""
    seen = set()
    for shift in (-3.0, -2.8, -2.6, -2.4, -2.2, -2.0, 3.0):
        ref = first_iteration(rows, cols, shift, rho, 60, False)
        runs = [first_iteration(rows, cols, shift, rho, 60, True) for _ in range(3)]
        for got in runs:
            assert got[:5] == ref[:5], (shift, got[:5], ref[:5])
            assert np.array_equal(got[5], runs[0][5])
        assert rel_err(runs[0][5], ref[5]) <= 1e-12, shift
        seen.add(ref[2])
    assert {1, 2, 3} < seen and max(seen) > 14, seen
