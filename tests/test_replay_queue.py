"""The solve loop's queue of graph replays (replay.h, host code): two in flight
at every wait, one where the replay in flight is expected to be the last, and two
again once such an expectation was wrong; never more than the bound."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def queue(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("replay") / "replay_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I",
                        os.path.join(ROOT, "paper_2512_09642_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "replay_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def run(bound, last):
        out = subprocess.run([exe, str(bound), last], capture_output=True, text=True)
        assert out.returncode == 0, out.stdout
        return [int(v) for v in out.stdout.split()]
    return run


@pytest.mark.parametrize("bound,last,depth", [
    (1, "", [1]), (2, "", [2, 1]), (5, "00000", [2, 2, 2, 2, 1]), (5, "1", [2, 1, 2, 2, 1]),
    (6, "011", [2, 2, 1, 1, 2, 1]), (8, "01010", [2, 2, 1, 2, 1, 2, 2, 1]), (4, "1111", [2, 1, 1, 1])])
def test_depth(queue, bound, last, depth):
    assert queue(bound, last) == depth + [bound]
