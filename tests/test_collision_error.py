"""The collision's own quotients, roots, exponentials and logarithms
(csrc/ecr_math.hpp) are no further from 80-bit arithmetic than the same
formulas with the library's exp and expm1, IEEE quotients and IEEE roots.

Both sides see the same 2^21 inputs.  The mean errors are compared: that of
a class is known to about 0.1% (a spread of an ulp or so over 10^5 to 10^6
inputs), the few inputs where 1 + u em cancels to about 1%, as the errors
there have a long tail.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1507_03392_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_errors_no_larger_than_the_plain_formulas(tmp_path):
    exe = str(tmp_path / "collision_error")
    subprocess.run(["g++", "-O2", "-std=c++20", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(HERE, "hostcheck", "collision_error.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=120).stdout
    rows = {w[0]: [float(v) for v in w[1:]] for w in map(str.split, out.splitlines())}
    assert set(rows) == {"s", "A<0.01", "A<0.35", "A<2", "A<20", "A>=20", "cancelling", "quotient"}
    for name, (n, mean, top, plain_mean, plain_top) in rows.items():
        assert n > 50_000, name
        assert mean <= plain_mean * (1.01 if name == "cancelling" else 1.001), (name, mean, plain_mean)
    # one rounding: the binary32-mixed s is as good as the IEEE quotient
    assert rows["quotient"][2] <= 0.5 + 2.0**-20
