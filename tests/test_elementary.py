"""log and log1p of the kernels (csrc/elementary.h, also compiled for the host): error below 0.6 units in the last place (0.5 from
the last rounding, at most 0.08 from the terms of up to 1 % of the result, each of a few roundings) over ranges that cover what the
entropy and logistic kernels ask for, and the values at the ends of the range.  On the device: test_gpu_elementary.py."""
import math
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def output(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("elementary") / "driver")
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=off", "-I", os.path.join(HERE, "..", "paper_2203_16340_amd", "csrc"),
                    os.path.join(HERE, "elementary", "driver.cpp"), "-o", exe], check=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()


def test_errors(output):
    lines = [line.split() for line in output if line.startswith("range")]
    assert len(lines) == 10
    for _, name, lo, hi, worst in lines:
        assert float(worst) <= 0.6, (name, lo, hi, worst)


def test_quotient(output):
    """Half a unit from the final rounding; the residue's correction leaves the square of the reciprocal's 2^-46."""
    assert float([line.split()[1] for line in output if line.startswith("quotient")][0]) <= 0.5000001


def test_special_values(output):
    lines = [[float(t) for t in line.split()[1:]] for line in output if line.startswith("at")]
    assert len(lines) == 9
    for x, log, log_ref, log1p, log1p_ref in lines:
        for got, ref in ((log, log_ref), (log1p, log1p_ref)):
            same = math.isnan(got) if math.isnan(ref) else (got == ref or abs(got - ref) <= 2.0 ** -52 * abs(ref))
            assert same, (x, got, ref)
