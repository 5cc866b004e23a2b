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
