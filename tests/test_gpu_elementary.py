"""log, log1p and the quotients of the logistic function as the kernels evaluate them on the device (lbfgsb_dbg_elementary),
against 80-bit arithmetic on the host.  The same code compiled for the host: test_elementary.py."""
import numpy as np
import pytest
import torch

import paper_2203_16340_amd as L
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

LOG, LOG1P, QUOTIENT_1, QUOTIENT_X = 0, 1, 2, 3
N = 400_000


def evaluate(which, x):
    xd = to_dev(x)
    y = torch.empty_like(xd)
    torch.cuda.synchronize()
    assert L.lib().lbfgsb_dbg_elementary(which, xd.numel(), xd.data_ptr(), y.data_ptr()) == L.OK
    return y.cpu().numpy()


def ulps(got, ref):
    """Largest distance from ref (long double) in units of the last place of a double."""
    _, e = np.frexp(ref.astype(np.float64))
    return float((np.abs(got.astype(np.longdouble) - ref) / np.ldexp(np.longdouble(1), e - 53)).max())


def arguments(lo, hi, logarithmic, seed):
    t = np.random.default_rng(seed).random(N)
    if not logarithmic:
        return lo + t * (hi - lo)
    sign = np.sign(lo)
    return sign * np.exp(np.log(sign * lo) + t * (np.log(sign * hi) - np.log(sign * lo)))


@pytest.mark.parametrize("lo,hi", [(1e-16, 1e-6), (-1e-16, -1e-6), (1e-9, 1e-7), (-1e-9, -1e-7)])
def test_log1p_of_small_arguments(lo, hi):
    """1 + x keeps few bits of x: what its rounding took away, divided by 1 + x, is as large as the result's last bits or larger."""
    x = arguments(lo, hi, True, 1)
    assert ulps(evaluate(LOG1P, x), np.log1p(x.astype(np.longdouble))) <= 0.6


@pytest.mark.parametrize("which,lo,hi,logarithmic", [
    (LOG, 0.5, 2.0, False), (LOG, 0.999, 1.001, False), (LOG, 1e-300, 1e300, True), (LOG, 1e-320, 1e-300, True),
    (LOG1P, -0.5, 1.0, False), (LOG1P, -0.999999, -0.4, False), (LOG1P, 1e-25, 1.0, True), (LOG1P, 1e-2, 1e200, True)])
def test_errors(which, lo, hi, logarithmic):
    """0.5 from the last rounding; beside it terms of at most 1 % of the result, with four roundings (and twice that of the square
    in the cube), so at most 0.08 and what the double-word sum leaves.  The runtime's functions reach 0.64."""
    x = arguments(lo, hi, logarithmic, 2)
    assert ulps(evaluate(which, x), (np.log if which == LOG else np.log1p)(x.astype(np.longdouble))) <= 0.6


@pytest.mark.parametrize("which", [QUOTIENT_1, QUOTIENT_X])
def test_quotients_are_correctly_rounded(which):
    rng = np.random.default_rng(3)
    x = np.concatenate([rng.random(N), np.exp(-700.0 * rng.random(N)), [0.0, 1.0, 5e-324]])
    np.testing.assert_array_equal(evaluate(which, x), (1.0 if which == QUOTIENT_1 else x) / (1.0 + x))


def test_ends_of_the_range():
    x = np.array([0.0, np.inf, -np.inf, np.nan, -1.0, -2.0, 1.0, 5e-324, np.finfo(np.float64).max])
    with np.errstate(divide="ignore", invalid="ignore"):
        np.testing.assert_allclose(evaluate(LOG, x), np.log(x), rtol=2.0 ** -52)
        np.testing.assert_allclose(evaluate(LOG1P, x), np.log1p(x), rtol=2.0 ** -52)


def test_refused():
    x = to_dev(np.ones(4))
    assert L.lib().lbfgsb_dbg_elementary(4, 4, x.data_ptr(), x.data_ptr()) == L.E_INVALID_ARG
    assert L.lib().lbfgsb_dbg_elementary(LOG, 0, x.data_ptr(), x.data_ptr()) == L.E_INVALID_ARG
    assert L.lib().lbfgsb_dbg_elementary(LOG, 4, None, x.data_ptr()) == L.E_INVALID_ARG
