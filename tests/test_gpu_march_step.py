"""The marched single basis step on both sides of its rule's lines (filled
unknowns, odd rows, what the step also writes): every column of a solver that takes
one step per launch equals the one of the two-step kernel bit for bit, and the
Gram matrix within the lockstep bar (1e-10; the FP32 one is formed from the same
columns by the same kernel)."""
import numpy as np
import pytest
import torch

import gen
from helpers import rel

pytestmark = pytest.mark.gpu

CASES = [((248, 180, 71), "fp64", "moments"), ((248, 180, 70), "fp64", "moments"), ((42, 31, 2450), "fp64", "moments"),
         ((39, 31, 2650), "fp64", "moments"),
         ((309, 180, 101), "fp64", "recurrence"), ((309, 180, 98), "fp64", "recurrence"),
         ((310, 180, 187), "fp64", "recurrence"), ((310, 180, 186), "fp64", "recurrence"),
         ((248, 180, 141), "fp32ir", "recurrence"), ((248, 180, 140), "fp32ir", "recurrence"),
         ((310, 180, 187), "fp64", "stored")]


@pytest.mark.parametrize("dims,precision,gram", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_columns_equal_pairs(hip, dims, precision, gram):
    lo, hi = gen.jacobi_poisson_bounds(*dims)
    n, s = int(np.prod(dims)), 3
    b = torch.rand(n, dtype=torch.float64, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(n))
    got = []
    for steps, gram in ((0, "recurrence" if gram == "stored" else gram), (1, gram)):
        with hip.Solver(hip.Operator.stencil(*dims), s, 10, lo, hi, precision=precision, gram=gram,
                        basis_steps=steps, autotune=False) as sv:
            got.append(sv.step(b, torch.zeros_like(b), want_basis=True))
    assert torch.equal(got[0]["P"], got[1]["P"])
    assert rel(got[0]["G"], got[1]["G"]) <= (1e-10 if precision == "fp64" else 0.0)
