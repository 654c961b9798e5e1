"""The choice of a factorisation's side stream, on the host: whatever goes wrong
after the first stream, that one serves."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1809_05334_amd", "csrc")


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("side") / "side_pick")
    p = subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=address,undefined", "-I", CSRC,
                        os.path.join(HERE, "side_pick.cpp"), "-o", exe], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    return lambda *a: [int(v) for v in subprocess.run([exe, *map(str, a)], capture_output=True, text=True,
                                                      check=True).stdout.split()]


@pytest.mark.parametrize("can,answers,want", [
    (9, [1], [1, 0, 0]),                       # the first runs beside: nothing is made
    (9, [0, 0, 1], [1, 2, 2, 0, 1]),           # the third does: the others go
    (9, [0, 0, 0, 0], [0, 0, 3, 1, 2, 3]),     # none does: the first stays
    (1, [0, 0], [0, 0, 1, 1]),                 # the third cannot be made: the first stays
    (0, [0], [0, 0, 0]),                       # no further one can be made
    (9, [-1], [0, 0, 0]),                      # no answer
    (9, [0, -1], [0, 0, 1, 1]),
])
def test_the_first_stream_serves_where_none_better_is_found(pick, can, answers, want):
    assert pick(can, 4, *answers) == want
