"""Two basis steps per launch of one large face-coefficient system, on both
sides of the lines of its rule (2^19 unknowns, bands that suit the grid) and where
its bands can go wrong: odd rows, rows of one point, one row of a band, a last
range of one plane, an odd count of columns, without Jacobi, the recurrence
kind.  One lockstep iteration against the oracle (1e-10), two outer iterations
against single steps (x within 1e-11: the same recurrence, products summed in
another order)."""
import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import make_operator, oracle_rhs, rel

pytestmark = pytest.mark.gpu

CASES = [((125, 17, 250), 4, True, "auto", 2), ((256, 64, 64), 5, True, "auto", 2), ((1, 1024, 513), 4, True, "auto", 2),
         ((1, 1025, 1024), 2, True, "auto", 1), ((7, 300, 251), 4, False, "auto", 2), ((83, 81, 80), 3, True, "recurrence", 1),
         ((128, 64, 64), 4, True, "auto", 2), ((128, 64, 63), 4, True, "auto", 0), ((257, 64, 33), 4, True, "auto", 0),
         ((200, 2700, 1), 2, True, "auto", 0), ((16, 16, 2100), 2, True, "auto", 0)]


@pytest.mark.parametrize("dims,s,precond,gram,pairs", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_face_bands(hip, dims, s, precond, gram, pairs):
    pr = gen.small_faces3d(*dims, seed=4, sigma=0.7, s=s, nu=15)
    A, b = oracle_rhs(pr)
    op = make_operator(hip, pr, "stencil")
    bt = torch.as_tensor(b, device="cuda:0")
    lo, hi = (pr.lmin, pr.lmax) if precond else (0.0, 2.0 * float(np.abs(A.diagonal()).max()) if hasattr(A, "diagonal") else 40.0)
    kw = dict(max_outer=2, precond=precond, gram=gram)
    with hip.Solver(op, s, 15, lo, hi, **kw) as sv:
        assert sv.basis_pairs == pairs
        x = torch.zeros_like(bt)
        g = sv.step(bt, x)
        o = oracle.step(A, b, np.zeros(pr.n), s, 15, lo, hi, precond=1 if precond else 0)
        for key in ("G", "ctil", "atil"):
            assert rel(g[key], o[key]) <= 1e-10, key
        assert rel(x.cpu().numpy(), o["x"]) <= 1e-10
        two, st2 = sv.solve(bt, None, 1e-15, raise_on_error=False)
    with hip.Solver(op, s, 15, lo, hi, basis_steps=1, **kw) as sv:
        assert sv.basis_pairs == 0
        one, st1 = sv.solve(bt, None, 1e-15, raise_on_error=False)
    assert st2.outer_iters == st1.outer_iters == 2
    assert rel(two.cpu().numpy(), one.cpu().numpy()) <= 1e-11
