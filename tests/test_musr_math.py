"""The quotient and the logarithm inside the fit statistic (csrc/musr_math.h),
run on the host against long double, with a reciprocal estimate of 22 bits.

Bounds, in units of the last place of the result.  Quotient: the corrected
product errs from the rounded quotient only where the remainder's own rounding
(2^-53 of a unit) decides, so 0.5 and a thousandth.  Logarithm: half a unit
for the last addition; the series beside it is at most 0.01 of the leading
term and carries a few roundings of itself (0.04 to 0.08 of a unit), and the
polynomial is off by 0.04: 0.65 in all, and a uniform rounding's 0.289 plus
these for the root mean square (below 0.30).  The device library's logarithm
measures 0.63 and 0.291 on ratios from 1/4 to 4."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def errors(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("musr_math") / "musr_math")
    subprocess.run([gxx, "-std=c++17", "-O2", "-ffp-contract=off", "-Wall", "-I",
                    os.path.join(ROOT, "paper_1509_07685_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "musr_math.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return {name: (float(worst), float(rms)) for name, worst, rms in (line.split() for line in out.splitlines())}


@pytest.mark.parametrize("name", ["quotient_counts", "quotient_all"])
def test_quotient_is_rounded_like_a_division(errors, name):
    worst, rms = errors[name]
    assert worst <= 0.501 and rms <= 0.29


@pytest.mark.parametrize("name", ["log_near_one", "log_ratio", "log_all"])
def test_logarithm_errs_no_more_than_the_library(errors, name):
    worst, rms = errors[name]
    assert worst <= 0.65 and rms <= 0.30


def test_exact_cases(errors):
    assert errors["log_one"][0] == 0.0
    assert errors["zero_divisor"][0] <= 1e-15      # n * 1/2 + n / 2, of 3.7
