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
