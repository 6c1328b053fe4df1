"""What the batched set-up's tuner times.  With the moments kind no launch of an
iteration depends on the tile schedule: nothing is timed, the default schedule
stays and the cache holds it as not measured.  With the other kinds a schedule is
chosen by the launches that depend on it, under a key that names them: an entry
that an earlier library wrote for other launches is not read."""
import json

import pytest
import torch

import gen

pytestmark = pytest.mark.gpu

SIDES = [104, 100]  # 2.1 million unknowns
SCHEMA = "sstep-tune-v2"


def batch(hip, **kw):
    ops = [hip.Operator.stencil(n, n, n) for n in SIDES]
    lo, hi = zip(*[gen.jacobi_poisson_bounds(n, n, n) for n in SIDES])
    return hip.BatchedSolver(ops, 1, 4, 10, lo, hi, **kw)


def key(kind, timed):
    h = 1469598103934665603
    for n in SIDES:
        h = ((h ^ n ** 3) * 1099511628211) % 2 ** 64
    return (f"{SCHEMA} gfx950 batched s=4 prec=fp64 nrhs=1 nsys=2 faces=0 rec=1 mom={int(kind == 'moments')} f2=1 "
            f"timed={timed} sizes={h:x}")


def test_moments_times_nothing(hip, tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("SSTEP_TUNE_CACHE", str(path))
    torch.cuda.synchronize()
    for _ in range(2):
        with batch(hip) as bt:
            assert bt.gram_kind == "moments"
            assert dict(bt.tiles) == {"rows_per_tile": 2048, "grid_factor": 4}
    entries = json.loads(path.read_text())
    assert [v["us"] for v in entries.values()] == [0]


def test_an_older_entry_is_not_read(hip, tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("SSTEP_TUNE_CACHE", str(path))
    old = key("recurrence", "iteration")
    path.write_text('{\n  "%s": {"nbg": 3, "slab": 2304, "us": 7.5}\n}\n' % old)
    with batch(hip, gram="recurrence") as bt:
        first = dict(bt.tiles)
    assert first["rows_per_tile"] in (2048, 8192, 32768) and first["grid_factor"] in (2, 4, 8)
    entries = json.loads(path.read_text())
    assert old in entries and len(entries) == 2 and entries[old]["slab"] == 2304
    with batch(hip, gram="recurrence") as bt:
        assert dict(bt.tiles) == first
