"""Overlapped coarse sweeps (sweep l runs wavefront t at step t + 8 l) on the
GPU against the oracle's sequential sweeps: hierarchies of fewer wavefronts
than the lag of 8, numbers of sweeps around it, thin ones, and both sides of
the line between one block and a launch per step (unknowns times sweeps over
steps: 25 streamed, 56 formed).  The bar is the coarse solve's, 1e-10; a step
that ran too early or too late would see values of another sweep."""
import pytest
import torch

import gen
import oracle
from helpers import rel

pytestmark = pytest.mark.gpu

CASES = [((1, 1, 1), 3), ((2, 2, 2), 1), ((2, 3, 1), 9), ((1, 1, 30), 20), ((40, 1, 1), 11), ((6, 6, 6), 2),
         ((7, 7, 7), 20), ((7, 7, 8), 30), ((9, 8, 9), 20), ((12, 11, 13), 5), ((16, 3, 9), 40)]


@pytest.mark.parametrize("nc,nu", CASES)
@pytest.mark.parametrize("formed", [False, True])
def test_overlapped_sweeps_equal_sequential(hip, nc, nu, formed):
    tl = gen.two_level(sum(nc) + nu, nc=nc, sigma=1.0, nu=nu)
    want, _ = oracle.coarse_fgs(tl.nc, tl.kx, tl.ky, tl.kz, tl.f, nu)
    op = hip.Operator.stencil(*tl.nf, tl.kx, tl.ky, tl.kz)
    f = torch.as_tensor(tl.f, device="cuda:0")
    with hip.CoarseSolver(op, formed=formed) as cs:
        first = cs.fgs(f, nu)
        again = cs.fgs(f, nu)
    assert rel(first.cpu().numpy(), want) <= 1e-10
    assert torch.equal(first, again)


# long thin hierarchies walked by one block whose tables do not fit the LDS: more
# than 1023 wavefronts, more than 4096 unknowns, both; and the same line again
LONG = [((1, 1, 300), 1), ((1, 1, 300), 8), ((1, 1, 300), 9), ((1030, 1, 1), 4), ((2, 1, 700), 3), ((5000, 1, 1), 2), ((17, 17, 17), 1),
        ((3, 40, 40), 1), ((1, 256, 1), 30)]


@pytest.mark.parametrize("nc,nu", LONG)
@pytest.mark.parametrize("formed", [False, True])
def test_long_hierarchies(hip, nc, nu, formed):
    test_overlapped_sweeps_equal_sequential(hip, nc, nu, formed)
