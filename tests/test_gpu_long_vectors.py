"""The checks of bounds, start point and gradient run on the device, four entries per thread and sweep, at most 1024
workgroups: an offending entry anywhere in a vector longer than one sweep (2^20 entries), in its clamped tail and at its
ends is found and named, and nothing of the solver's state has changed."""
import numpy as np
import pytest
import torch

import paper_2203_16340_amd as L
from gpu_helpers import DEV, to_dev

pytestmark = pytest.mark.gpu

N = (1 << 20) + 4099
PLACES = [0, (1 << 20) - 1, 1 << 20, (1 << 20) + 2500, N - 1]


def _parts():
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1)
    A = torch.rand(2, N, dtype=torch.float64, device=DEV, generator=gen)
    b = torch.ones(2, dtype=torch.float64, device=DEV)
    l = torch.zeros(N, dtype=torch.float64, device=DEV)
    u = torch.full((N,), 2.0, dtype=torch.float64, device=DEV)
    return A, b, l, u


def _code(call):
    with pytest.raises(L.LbfgsbError) as e:
        call()
    return e.value.code, str(e.value)


@pytest.mark.parametrize("place", PLACES)
@pytest.mark.parametrize("uniform", [True, False])
def test_start_point(place, uniform):
    A, b, l, u = _parts()
    if not uniform:
        u[7] = 3.0
    s = L.Solver(L.OBJ_LSQ, A, b, l, u, 3)
    good = torch.full((N,), 1e-6, dtype=torch.float64, device=DEV)
    s.set_x(good)
    before = s.info().as_dict()
    for bad in (-1e-300, 5.0, float("nan")):
        x0 = good.clone()
        x0[place] = bad
        code, message = _code(lambda: s.set_x(x0))
        assert code == L.E_INFEASIBLE_X0 and f"x0[{place}]" in message
    assert s.info().as_dict() == before and torch.equal(s.x(), good)
    s.set_x(torch.where(torch.arange(N, device=DEV) == place, u, good))      # (on the bound is inside)
    s.close()


@pytest.mark.parametrize("place", PLACES)
def test_bounds(place):
    A, b, l, u = _parts()
    for lo, hi in ((3.0, 2.0), (float("nan"), 2.0), (0.0, float("nan"))):
        bad_l, bad_u = l.clone(), u.clone()
        bad_l[place], bad_u[place] = lo, hi
        code, message = _code(lambda: L.Solver(L.OBJ_LSQ, A, b, bad_l, bad_u, 3))
        assert code == L.E_BOUNDS and f"index {place}" in message
    # a single pair that differs is seen: its variable stays inside its own bounds
    tight = u.clone()
    tight[place] = 1e-9
    s = L.Solver(L.OBJ_LSQ, A, b, l, tight, 3, options=L.default_options(max_iter=3))
    s.set_x(l)
    s.solve()
    x = s.x()
    assert 0.0 <= float(x[place]) <= 1e-9 and float(x.max()) > 1e-9
    s.close()


@pytest.mark.parametrize("place", PLACES)
def test_entropy_needs_positive_lower_bounds(place):
    rows, cols = 1025, 1027                                                  # 1 052 675 entries
    place = min(place, rows * cols - 1)
    M = torch.ones(rows, cols, dtype=torch.float64, device=DEV)
    l = torch.full((rows * cols,), 1e-20, dtype=torch.float64, device=DEV)
    u = torch.full((rows * cols,), 1.0, dtype=torch.float64, device=DEV)
    l[place] = 0.0
    code, message = _code(lambda: L.Solver(L.OBJ_OT_ENTROPY, M, None, l, u, 3, lam=0.5))
    assert code == L.E_BOUNDS and f"l[{place}]" in message


@pytest.mark.parametrize("place", PLACES)
def test_gradient_that_is_not_finite(place):
    """f = 0.5 (1e100)^2 is finite, the gradient's entry 1e250 * 1e100 is not."""
    A, b, l, u = _parts()
    A[0, place] = 1e250
    b[0] = -1e100
    s = L.Solver(L.OBJ_LSQ, A, b, l, u, 3)
    assert _code(lambda: s.set_x(l))[0] == L.E_NONFINITE
    s.close()
