"""Operator arrays in device memory, written by work that is still running on
the caller's stream when the set-up or the update is called: the library reads
them after that work, whatever stream it is on."""
import numpy as np
import pytest
import torch

import gen

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def late(values, stream):
    """Device copies of values that appear behind other work on stream."""
    out = [torch.full((v.size,), float("nan"), dtype=torch.float64, device=DEV) for v in values]
    src = [torch.as_tensor(np.ascontiguousarray(v), device=DEV) for v in values]
    a = torch.ones(3000, 3000, dtype=torch.float64, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(20):
            a = a @ a * 1e-4
        for o, s in zip(out, src):
            o.copy_(s)
    return out


@pytest.mark.parametrize("side", [False, True])
def test_faces_written_on_the_callers_stream(hip, side):
    pr = gen.small_faces3d(30, 27, 25, seed=1, sigma=0.5)
    b = torch.as_tensor(gen.uniform(gen.rng(2), pr.n), device=DEV)
    stream = torch.cuda.Stream() if side else torch.cuda.current_stream()
    kw = dict(max_outer=3, stream=stream)
    faces, other = [pr.kx, pr.ky, pr.kz], [2.0 * k + 1.0 for k in (pr.kx, pr.ky, pr.kz)]
    want = []
    for f in (faces, other):  # from host arrays
        with hip.Solver(hip.Operator.stencil(*pr.dims, *f), 8, 20, 0.0, 2.0, max_outer=3) as sv:
            want.append(sv.solve(b, None, 1e-12, raise_on_error=False)[0])
    with hip.Solver(hip.Operator.stencil(*pr.dims, *late(faces, stream)), 8, 20, 0.0, 2.0, **kw) as sv:
        assert torch.equal(sv.solve(b, None, 1e-12, raise_on_error=False)[0], want[0])
        sv.update_coefficients(hip.Operator.stencil(*pr.dims, *late(other, stream)))
        assert torch.equal(sv.solve(b, None, 1e-12, raise_on_error=False)[0], want[1])


def test_faces_written_on_the_default_stream(hip):
    """A solver on a stream of its own, the arrays from the default stream: the
    set-up, the update, a batch and a coarse solver read them after that too."""
    pr = gen.small_faces3d(31, 27, 25, seed=4, sigma=0.5)
    b = torch.as_tensor(gen.uniform(gen.rng(2), pr.n), device=DEV)
    side, default = torch.cuda.Stream(), torch.cuda.default_stream()
    faces, other = [pr.kx, pr.ky, pr.kz], [2.0 * k + 1.0 for k in (pr.kx, pr.ky, pr.kz)]
    nc = (15, 13, 12)
    f = torch.as_tensor(gen.uniform(gen.rng(3), int(np.prod(nc))), device=DEV)
    torch.cuda.synchronize()
    got = []
    for place in (lambda v: v, lambda v: late(v, default)):
        with hip.Solver(hip.Operator.stencil(*pr.dims, *place(faces)), 8, 20, 0.0, 2.0, max_outer=3, stream=side) as sv:
            x = [sv.solve(b, None, 1e-12, raise_on_error=False)[0]]
            sv.update_coefficients(hip.Operator.stencil(*pr.dims, *place(other)))
            x.append(sv.solve(b, None, 1e-12, raise_on_error=False)[0])
        with hip.BatchedSolver([hip.Operator.stencil(*pr.dims, *place(faces))], 1, 8, 20, [0.0], [2.0], max_outer=3,
                               stream=side) as bt:
            x.append(bt.solve([b], None, 1e-12, raise_on_error=False)[0][0])
        with hip.CoarseSolver(hip.Operator.stencil(*pr.dims, *place(faces)), stream=side) as cs:
            x.append(cs.fgs(f, 3))
        torch.cuda.synchronize()
        got.append(x)
    for a, c in zip(*got):
        assert torch.equal(a, c)
