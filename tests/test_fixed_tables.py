"""The lattice-sum coefficients of the mixed-precision operator, to the bit.

Its far entries are rounded to FP32, so a coefficient that differs in its last
bit moves isolated entries of Z to the neighbouring FP32 value and a component
of the solution by up to 1e-7.  The digests below (one per cell and incidence)
hold every coefficient of the fixed evaluation."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1809_05334_amd", "csrc")

DIGESTS = {   # (a, b, zspan, lambda, theta, phi)
    (100, 100, 50, 600, 0.4, 0.3): "3b7e749c034ca4b1",
    (157, 157, 114, 612, 0.5, 0.7): "d36d7156a4d94fa0",
    (157, 120, 114, 650, 0, 0): "7911bab3b6066187",
    (200, 200, 120, 555, 0.8, 0.2): "79fed3f43b066a3e",
    (60, 60, 100, 480, 0.3, 1.1): "953e7c1d414e6521",
    (300, 240, 90, 400, 0.7, 0.3): "de46c0bdf9beca10",
}


def test_coefficients_are_the_recorded_ones(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path / "fixed_tables")
    p = subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-I", os.path.join(os.path.dirname(HERE), "include"),
                        os.path.join(HERE, "fixed_tables.cpp"), os.path.join(CSRC, "tables.cpp"), "-o", exe, "-lpthread"],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    inp = "\n".join(" ".join(map(str, k)) for k in DIGESTS)
    p = subprocess.run([exe], input=inp, capture_output=True, text=True, timeout=120)
    assert p.returncode == 0
    assert p.stdout.split() == list(DIGESTS.values())
