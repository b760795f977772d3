"""Both replays of the contracted walk (parent pointers within their budget,
the labelled forest beyond it) against the one-by-one walk; built with address
and undefined-behaviour sanitizers (host code only)."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def binary():
    exe = os.path.join(tempfile.mkdtemp(), "replay_check")
    subprocess.check_call([
        "g++", "-O1", "-g", "-std=c++17", "-pthread", "-fsanitize=address,undefined",
        "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "paper_2509_14433_amd", "csrc"),
        os.path.join(ROOT, "tests", "native", "replay_check.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("V,m,n,seed,path", [(6000, 900, 6000, 1, 1), (3000, 2500, 9000, 2, 1),
                                             (6000, 900, 6000, 3, 0), (50, 10, 4000, 4, 1),
                                             (4000, 3000, 3000, 5, 0)])
def test_replays_match_one_by_one(binary, V, m, n, seed, path):
    r = subprocess.run([binary, str(V), str(m), str(n), str(seed), str(path)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    # an insert on a path of hundreds of pieces walks far more than 64 of them
    assert r.stdout == f"labelled={int(path and m > 500)}\n"
