"""Small batches on the GPU: the z-ranges shorter than 16 planes they take, the
Gram tiles whose rows load in groups (remainders of one to three steps, tiles
of a few rows), and the update by points, in batches of one pair to a few
dozen.  x after two outer iterations equals one basis step per launch bit for
bit (recurrence kind), FP64 and FP32, widths on both sides of the Gram's column
blocks; FP64 against the oracle at 1e-10."""
import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,nrhs,s", [
    ([(5, 4, 3)], 1, 2), ([(16, 16, 8), (16, 16, 9)], 1, 8), ([(13, 13, 13), (11, 30, 20), (33, 33, 33)], 3, 8),
    ([(9, 9, 9), (17, 16, 15), (40, 40, 2)], 5, 16), ([(20, 20, 61)], 9, 17), ([(8, 8, 32)] * 12, 2, 4)])
@pytest.mark.parametrize("precision", ["fp64", "fp32ir"])
def test_small_batch(hip, dims, nrhs, s, precision):
    r = gen.rng(21)
    lo, hi = gen.gershgorin_jacobi_bounds()
    faces = [gen.face_coefficients(r, *d, 1.0) for d in dims]
    rhs = [np.stack([gen.uniform(r, int(np.prod(d))) for _ in range(nrhs)]) for d in dims]
    ops = [hip.Operator.stencil(*d, *k) for d, k in zip(dims, faces)]
    got = []
    for steps in (0, 1):
        with hip.BatchedSolver(ops, nrhs, s, 20, [lo] * len(ops), [hi] * len(ops), max_outer=2, autotune=False,
                               gram="recurrence", precision=precision, basis_steps=steps) as bs:
            x, st = bs.solve([torch.as_tensor(b.ravel(), device="cuda:0") for b in rhs], None, 1e-15,
                             raise_on_error=False)
        got.append([v.cpu().numpy().reshape(nrhs, -1) for v in x])
    for q, (d, k) in enumerate(zip(dims, faces)):
        assert np.array_equal(got[0][q], got[1][q]), (d, rel(got[0][q], got[1][q]))
        if precision == "fp64" and s <= 8:
            A = oracle.assemble_stencil7(*d, *k)
            for p in range(nrhs):
                x = np.zeros(rhs[q].shape[1])
                for _ in range(2):
                    x = oracle.step(A, rhs[q][p], x, s, 20, lo, hi)["x"]
                assert rel(got[0][q][p], x) <= 1e-10, (d, p)
