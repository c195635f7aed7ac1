"""GELU and its derivative as the training kernel evaluates them (gelu_both),
compiled for the host: against 64 bits no further off than with erff and
expf, in the worst case and on average, over the inputs of a trained network
and out to where both are flat; infinities and NaN come out as with erff."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("gelu") / "check")
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=off", "-std=c++17",
                    "-I", os.path.join(ROOT, "paper_2005_13498_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "gelu_check.cpp"), "-o", exe], check=True)

    def f(lo, hi):
        out = subprocess.run([exe, str(lo), str(hi), "2000001"], capture_output=True, text=True, check=True, timeout=60)
        return [[float(x) for x in line.split()] for line in out.stdout.strip().splitlines()]
    return f


@pytest.mark.parametrize("lo,hi", [(-8, 8), (-2, 2), (-1, 1), (0.5, 4), (-4, -0.5)])
def test_errors_are_no_larger_than_with_erff(check, lo, hi):
    h, d, he, de, special = check(lo, hi)
    # (5 %: the last point may fall on the other side of a rounding)
    assert h[0] <= he[0] * 1.05 and h[1] <= he[1] * 1.05
    assert d[0] <= de[0] * 1.05 and d[1] <= de[1] * 1.05
    assert special == [1, 1, 1, 1]
