"""Grids of more blocks than one launch takes: the update of a batch in several
launches (more than 2^21 blocks of 256 points and right-hand side), and a thin
grid whose bricks would be too many (2^22 blocks of 1024 threads) and which marches
instead."""
import pytest
import torch

import gen
from helpers import rel

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_update_in_several_launches(hip):
    """40 equal right-hand sides of 240^3: 2.16 million blocks.  Every iterate is
    the first one, which is a batch's of one pair (FP32 columns, summed over
    other bands: 1e-5)."""
    n, nrhs = 240, 40
    assert -(-n ** 3 // 256) * nrhs > 2 ** 21
    lo, hi = gen.jacobi_poisson_bounds(n, n, n)
    op = hip.Operator.stencil(n, n, n)
    b = torch.rand(n ** 3, dtype=torch.float64, device=DEV)
    kw = dict(precision="fp32ir", max_outer=1, autotune=False)
    with hip.BatchedSolver([op], nrhs, 2, 10, [lo], [hi], **kw) as bt:
        x, st = bt.solve([b.repeat(nrhs)], None, 1e-12, raise_on_error=False)
    x = x[0].view(nrhs, -1)
    assert all((v.outer_iters, v.rel_res) == (1, st[0].rel_res) for v in st)
    assert all(torch.equal(x[r], x[0]) for r in range(nrhs))
    with hip.BatchedSolver([op], 1, 2, 10, [lo], [hi], **kw) as one:
        y, _ = one.solve([b], None, 1e-12, raise_on_error=False)
    assert rel(x[0].cpu().numpy(), y[0].cpu().numpy()) <= 1e-5


def test_bricks_too_many_for_a_launch(hip):
    """11 x 12 points a plane, 264 to a brick: one plane's worth on either side of
    2^22 bricks.  The iterate of x-y-constant data far from the ends is the one of
    a short grid."""
    s, planes = 2, 3 * 2 ** 20
    free, _ = torch.cuda.mem_get_info()
    if free < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    got = []
    for nz in (6000, 2 * 2 ** 22 + 2):
        assert nz == 6000 or nz > planes
        lo, hi = gen.jacobi_poisson_bounds(11, 12, 6000)
        n = 11 * 12 * nz
        with hip.Solver(hip.Operator.stencil(11, 12, nz), s, 5, lo, hi, max_outer=1) as sv:
            assert sv.basis_pairs == 1
            x, st = sv.solve(torch.ones(n, dtype=torch.float64, device=DEV), None, 1e-12, raise_on_error=False)
        assert st.outer_iters == 1
        x = x.view(nz, 132)
        got.append((x[:20].clone(), x[-20:].clone(), x[nz // 2].clone(), st.rel_res))
        del x
    for v in got[1][:2]:
        assert bool(torch.isfinite(v).all())
    # both ends mirror each other, and the middle is the one of the short grid up to
    # what the ends weigh in the coefficients (1 / 6000)
    assert rel(got[1][0].cpu().numpy(), got[1][1].flip(0).cpu().numpy()) <= 1e-12
    assert rel(got[1][2].cpu().numpy(), got[0][2].cpu().numpy()) <= 1e-2
    assert abs(got[1][3] - got[0][3]) <= 1e-2 * got[0][3]
