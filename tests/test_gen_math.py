"""The generator's binary64 functions (csrc/kb_math.hpp) on the host, against
80-bit long double at the ends of every reduction interval and on a million
spread words, with seeds twice as far off as the device's instructions may be.

Bounds, in units in the last place of binary64, from the roundings each
result passes (half a unit each): -2 ln u five (the quotient two, the
polynomial's last step, its product, the sum with the exponent) and the
polynomial error of 2^-59; the square root two (its first product counts
half); sine and cosine the polynomial's last step, and the reduction's last
rounding scaled by at most tan or cot of pi / 4, with the neglected
polynomial roundings below a quarter of a unit each; the Student-t half of
the two logarithms' five units, the cosine's 1.5 and five roundings of its
own.  "edges" are the Student-t's values where a pair's u is 1."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BOUND = {"edges": 0.0, "student_t3": 6.0, "neg2_log": 2.6, "sqrt": 1.0, "sin": 1.5, "cos": 1.5}


def build(tmp_path):
    exe = str(tmp_path / "gen_math_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", os.path.join(ROOT, "tests", "gen_math_check.cpp"),
                    "-o", exe], check=True, capture_output=True, text=True)
    return exe


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_first_pass_interval_covers_its_errors(tmp_path):
    """The 16-bit normals' first pass: the binary32 normal is rho32 times a
    sine or cosine of sincos32, rounded once (one unit of 2^-24), and the
    definition's value must lie within a factor 1 -+ 1.25 * 2^-21 (10 units)
    of it; the roundings after that are monotone.  The errors are the largest
    over 70 million words, the logarithm and the root one unit in the last
    place off either way; 0.01 covers their second-order terms and the
    binary64 value's own error."""
    out = subprocess.run([build(tmp_path), "32"], check=True, capture_output=True, text=True, timeout=300).stdout
    lines = [l.split() for l in out.splitlines()]
    assert [l[0] for l in lines] == ["rho32", "sincos32", "rho32", "rho32"]
    err = [float(l[1]) for l in lines]
    assert err[0] <= 2.2 and err[1] <= 3.3, lines
    assert max(err[2:]) + err[1] + 1.0 + 0.01 < 1.25 * 2.0 ** -21 * 2.0 ** 24, lines


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_generator_math_against_long_double(tmp_path):
    exe = str(tmp_path / "gen_math_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", os.path.join(ROOT, "tests", "gen_math_check.cpp"),
                    "-o", exe], check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=300).stdout
    lines = [l.split() for l in out.splitlines()]
    assert [l[0] for l in lines] == list(BOUND) * 2
    for name, worst, at in lines:
        assert float(worst) <= BOUND[name], (name, worst, at)
