"""Two basis steps per launch at the edges of the kernel's tiles, on the GPU.

A block's extended tile is 64 x 32 points: an axis that fits with its ring (62
points along x, 30 along y) is one tile, a longer one is cut into tiles of at
most 60 x 28.  The grids sit on both sides of those lines, with ranges of few
and many planes.  A pair forms each value with the operations of a single step
in the same order, so every basis column equals the one of a solver that takes
one step per launch bit for bit; the Gram matrix differs in the order of its
sums only (the lockstep bar, 1e-10)."""
import numpy as np
import pytest
import torch

import gen
from helpers import rel

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

SEVEN = [(62, 30, 5), (63, 31, 4), (60, 28, 9), (61, 29, 1), (64, 57, 3), (121, 33, 2), (1, 1, 7), (2, 90, 6),
         (125, 3, 40)]
# the 27-point operator takes pairs from 327680 unknowns on
BOX = [(62, 30, 177), (63, 31, 168), (121, 57, 48), (300, 400, 3), (64, 64, 81)]


@pytest.mark.parametrize("precision", ["fp64", "fp32ir"])
@pytest.mark.parametrize("op,dims", [("7", d) for d in SEVEN] + [("27", d) for d in BOX])
def test_pair_columns_equal_single_steps(hip, op, dims, precision):
    if op == "7":
        mk, (lo, hi) = hip.Operator.stencil, gen.jacobi_poisson_bounds(*dims)
    else:
        mk, (lo, hi) = hip.Operator.stencil27, gen.jacobi_poisson27_bounds(*dims)
    n, s = int(np.prod(dims)), 5
    b = torch.as_tensor(gen.uniform(gen.rng(n), n), device=DEV)
    got = []
    for steps in (0, 1):
        with hip.Solver(mk(*dims), s, 10, lo, hi, precision=precision, basis_steps=steps, autotune=False) as sv:
            assert sv.basis_pairs == (s // 2 if steps == 0 else 0)
            x = torch.zeros_like(b)
            try:
                got.append(sv.step(b, x, want_basis=True))
            except hip.SStepError:  # a grid with fewer eigenvectors than columns breaks down, both ways
                got.append(None)
    assert (got[0] is None) == (got[1] is None)
    if got[0] is not None:
        assert torch.equal(got[0]["P"], got[1]["P"])
        assert rel(got[0]["G"], got[1]["G"]) <= (1e-10 if precision == "fp64" else 0.0)
