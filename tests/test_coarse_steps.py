"""The launches of the overlapped coarse sweeps (coarse_steps.h, host code): every
sweep takes every wavefront once, at step t + 8 l, and a step of a long thin
hierarchy with many sweeps goes in launches of at most 65535 block rows."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("coarse") / "coarse_steps_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I",
                        os.path.join(ROOT, "paper_2512_09642_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "coarse_steps_check.cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("nwf,nu", [(1, 1), (1, 5), (7, 1), (8, 3), (9, 3), (113, 1), (113, 20), (16, 40), (2000, 300)])
def test_every_wavefront_of_every_sweep(exe, nwf, nu):
    r = subprocess.run([exe, str(nwf), str(nu), "1"], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
    steps, launches, most = [int(v) for v in r.stdout.split()]
    # fewer than 8 wavefronts leave steps without any
    assert steps == nwf + 8 * (nu - 1) and launches == (steps if nwf >= 8 else nwf * nu)
    assert most <= min(nu, (nwf + 7) // 8)


def test_more_rows_than_a_launch_holds(exe):
    """1 x 1 x 150000 unknowns, 80000 sweeps, some of the steps."""
    r = subprocess.run([exe, str(1 + 2 + 4 * 150000 - 6), "80000", "49999"], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
    assert [int(v) for v in r.stdout.split()][2] == 65535
