"""A solve whose initial guess is not finite stops with SSTEP_E_NONFINITE and
leaves nothing behind: the iterate it staged in LDS stays there until another
kernel overwrites it, and the two-step face kernel (band_f2.h), which sums products
of every value it forms, must not read such a value.  After solves that fill the
LDS of the whole chip with NaN, a large face-coefficient system (bands of its rows)
and the healthy pairs of a batch end as in single steps, which keep no plane in
LDS: the same iteration count and status, x within 1e-11 (the same recurrence,
products summed in another order)."""
import numpy as np
import pytest
import torch

import gen
from helpers import rel

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def t64(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)


@pytest.fixture(scope="module")
def nan_everywhere(hip):
    """Runs a solve that marches a vector of NaN through LDS on every CU."""
    n = 192
    lo, hi = gen.jacobi_poisson_bounds(n, n, n)
    b = torch.ones(n ** 3, dtype=torch.float64, device=DEV)
    with hip.Solver(hip.Operator.stencil(n, n, n), 2, 5, lo, hi) as sv:
        def run():
            _, st = sv.solve(b, torch.full_like(b, float("nan")), 1e-8, raise_on_error=False)
            assert (st.outer_iters, st.status) == (0, 6)
        yield run


@pytest.mark.parametrize("gram", ["moments", "recurrence"])
def test_large_face_system(hip, nan_everywhere, gram):
    dims, s = (128, 64, 64), 4
    r = gen.rng(7)
    lo, hi = gen.gershgorin_jacobi_bounds()
    op = hip.Operator.stencil(*dims, *gen.face_coefficients(r, *dims, 0.7))
    b = t64(gen.uniform(r, int(np.prod(dims))))
    got = []
    for steps in (0, 1):
        with hip.Solver(op, s, 15, lo, hi, max_outer=2, gram=gram, basis_steps=steps) as sv:
            assert sv.basis_pairs == (0 if steps else s // 2)
            nan_everywhere()
            x, st = sv.solve(b, None, 1e-15, raise_on_error=False)
            got.append((x.cpu().numpy(), st.outer_iters, st.status))
    assert got[0][1:] == got[1][1:] == (2, 5)
    assert rel(got[0][0], got[1][0]) <= 1e-11


@pytest.mark.parametrize("faces", [True, False], ids=["faces", "const"])
def test_batch_with_nonfinite_starts(hip, nan_everywhere, faces):
    """Half the pairs of every system start from NaN, the other half from
    zero."""
    dims, nrhs, s = [(40, 38, 36), (33, 35, 34), (64, 20, 40)], 8, 8
    r = gen.rng(9)
    ops, lo, hi, b, x0 = [], [], [], [], []
    for d in dims:
        n = int(np.prod(d))
        ops.append(hip.Operator.stencil(*d, *(gen.face_coefficients(r, *d, 1.0) if faces else ())))
        bounds = gen.gershgorin_jacobi_bounds() if faces else gen.jacobi_poisson_bounds(*d)
        lo.append(bounds[0])
        hi.append(bounds[1])
        b.append(t64(gen.uniform(r, n * nrhs)))
        v = torch.zeros(nrhs, n, dtype=torch.float64, device=DEV)
        v[::2] = float("nan")
        x0.append(v.reshape(-1))
    got = []
    for steps, gram in ((0, "moments"), (1, "recurrence")):
        with hip.BatchedSolver(ops, nrhs, s, 20, lo, hi, max_outer=2, gram=gram, basis_steps=steps,
                               autotune=False) as bt:
            for _ in range(2):
                nan_everywhere()
                x, st = bt.solve(b, [v.clone() for v in x0], 1e-15, raise_on_error=False)
            got.append(([v.cpu().numpy().reshape(nrhs, -1) for v in x], [(v.outer_iters, v.status) for v in st]))
    assert got[0][1] == got[1][1] == [(0, 6), (2, 5)] * (nrhs // 2 * len(dims))
    for q in range(len(dims)):
        for k in range(1, nrhs, 2):
            assert rel(got[0][0][q][k], got[1][0][q][k]) <= 1e-11, (q, k)
