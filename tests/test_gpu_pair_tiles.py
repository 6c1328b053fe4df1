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
import oracle
from helpers import make_operator, oracle_rhs, rel

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


# grids that take the marched residual (327680 unknowns) and the marched single
# step (27-point: 524288, 7-point: 3145728), at the edges of its 62 x 30 tiles
MARCHED = [("7", (62, 30, 177)), ("7", (63, 31, 169)), ("7", (186, 181, 94)), ("27", (64, 65, 127)),
           ("27", (61, 31, 280)), ("27", (125, 92, 46)), ("27", (380, 700, 2))]


@pytest.mark.parametrize("op,dims", MARCHED)
def test_marched_residual_and_step_lockstep(hip, op, dims):
    """One step per launch (three columns) against the oracle at the lockstep
    bars: residual norm and columns 1e-12, G, ctil, atil and x 1e-10."""
    pr = (gen.small_poisson3d if op == "7" else gen.small_poisson27)(*dims, seed=sum(dims), s=3, nu=10)
    A, b = oracle_rhs(pr)
    bt = torch.as_tensor(b, device=DEV)
    x = np.zeros(pr.n)
    with hip.Solver(make_operator(hip, pr, "stencil"), 3, 10, pr.lmin, pr.lmax, basis_steps=1) as sv:
        for k in range(2):
            xt = torch.as_tensor(x, device=DEV)
            g = sv.step(bt, xt, want_basis=True)
            o = oracle.step(A, b, x, 3, 10, pr.lmin, pr.lmax, want_basis=True)
            assert abs(g["rnorm"] - o["rnorm"]) <= 1e-12 * o["rnorm"]
            P = g["P"].cpu().numpy()
            for j in range(3):
                assert rel(P[j], o["P"][j]) <= 1e-12, (k, j)
            for key in ("G", "ctil", "atil"):
                assert rel(g[key], o[key]) <= 1e-10, (k, key)
            x = xt.cpu().numpy()
            assert rel(x, o["x"]) <= 1e-10, k
