"""Two basis steps per launch of one face-coefficient system, in bricks and in
bands, give every column bit for bit as one step per launch does (the promise of
the option basis_steps), with and without Jacobi, in both kinds that keep no A p;
the Gram matrix differs in the order of its sums only (the lockstep bar, 1e-10)."""
import numpy as np
import pytest
import torch

import gen
from helpers import rel

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [((16, 16, 8), 4), ((17, 9, 15), 6), ((1, 3000, 1), 4), ((64, 64, 64), 8), ((128, 64, 64), 5),
         ((125, 17, 250), 4), ((83, 81, 80), 3), ((1, 1024, 513), 4)]


@pytest.mark.parametrize("gram", ["moments", "recurrence"])
@pytest.mark.parametrize("precond", [True, False])
@pytest.mark.parametrize("dims,s", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_columns_equal_single_steps(hip, dims, s, precond, gram):
    r = gen.rng(3)
    op = hip.Operator.stencil(*dims, *gen.face_coefficients(r, *dims, 0.7))
    b = torch.as_tensor(gen.uniform(r, int(np.prod(dims))), device=DEV)
    got = []
    for steps in (0, 1):
        with hip.Solver(op, s, 10, 0.0, 2.0 if precond else 60.0, precond=precond, gram=gram, basis_steps=steps) as sv:
            assert sv.basis_pairs == (0 if steps else s // 2)
            got.append(sv.step(b, torch.zeros_like(b), want_basis=True))
    for j in range(s):
        assert torch.equal(got[0]["P"][j], got[1]["P"][j]), j
    assert rel(got[0]["G"], got[1]["G"]) <= 1e-10
