"""Short vectors: free set, Gram matrix, recursion, direction and Algorithm 2's choice in one workgroup, iteration by
iteration against the oracle at the edges of the kernel's sizes (waves of 64, rounds of 512, its widest n for m <= 5, 10,
20, and the first sizes left to the other kernels), through the first turns of the pair memory.

Bound: the two sides add the same k <= 1024 products in other orders (relative 1e-13 per sum), and a Gaussian problem with
four rows per column amplifies that by about ten per iteration while it converges; iterates are asked to 1e-8 over at most
12 iterations, decisions exactly."""
import numpy as np
import pytest

import oracle
import paper_2203_16340_amd as L
from gpu_helpers import make_solver, rel_err, to_dev

pytestmark = pytest.mark.gpu

SIZES = [(2, 3), (3, 1), (63, 5), (64, 5), (65, 5), (127, 4), (511, 5), (512, 5), (513, 5), (1023, 5), (1024, 5), (1025, 5),
         (63, 10), (65, 7), (200, 6), (511, 10), (512, 10), (513, 10), (831, 9), (832, 10), (833, 10),
         (65, 20), (130, 11), (383, 20), (384, 20), (385, 20), (100, 21)]


@pytest.mark.parametrize("n,m", SIZES)
@pytest.mark.parametrize("two_sided", [False, True])
def test_iterations_against_the_oracle(n, m, two_sided):
    rng = np.random.default_rng(1000 * n + m)
    rows = 4 * n + 260
    A = rng.standard_normal((rows, n)) / np.sqrt(rows)
    x_true = rng.standard_normal(n)
    b = A @ x_true + 0.1 * rng.standard_normal(rows)
    l = np.full(n, -0.4) if two_sided else np.zeros(n)
    u = np.full(n, 0.7) if two_sided else np.full(n, np.inf)
    x0 = np.clip(0.3 * rng.standard_normal(n), l, u)
    print(f"n {n} m {m} two_sided {two_sided}", flush=True)
    s = make_solver(L.OBJ_LSQ, A, b, l, u, m, tol=0.0, refresh_every=0)
    s.set_x(to_dev(x0))
    orc = oracle.Solver(oracle.Objective(L.OBJ_LSQ, A, b), l, u, x0, m, oracle.default_options(tol=0.0))
    for k in range(min(m + 3, 12)):
        if orc.step() != oracle.RUNNING or orc.info.pg2 < 1e-9:
            break                                           # (a handful of variables: at the solution)
        info = s.step()
        oi = orc.info
        assert info.status == L.RUNNING and info.iters == k + 1
        assert (info.branch, info.backtracks, info.pairs_used, info.n_fixed) == (oi.branch, oi.backtracks, oi.pairs_used, oi.n_fixed)
        assert info.pg2 == pytest.approx(oi.pg2, rel=1e-7)
        assert rel_err(s.x().cpu().numpy(), orc.x) <= 1e-8
    assert k >= 1 or n <= 3
