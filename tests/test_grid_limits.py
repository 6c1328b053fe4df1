"""Launches of more blocks than one may hold (grid_limits.h, host code): every
block in exactly one launch of fewer than 2^32 threads, a failure ends them."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches_cover_the_blocks(tmp_path):
    exe = str(tmp_path / "grid_limits_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I",
                        os.path.join(ROOT, "paper_2512_09642_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "grid_limits_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    blocks = [0, 1, 2 ** 21 - 1, 2 ** 21, 2 ** 21 + 1, 512 ** 3 // 256 * 32, 2 ** 32 - 1, 3 * 2 ** 32]
    out = subprocess.run([exe, *map(str, blocks)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    got = [[int(v) for v in line.split()] for line in out.stdout.splitlines()]
    assert got[:-1] == [[b, -(-b // 2 ** 21)] for b in blocks]
    assert got[-1] == [1, 0]
