"""Two basis steps per launch of a small 7-point system in bricks of 8^3
points: grids that fill the bricks, leave one plane, row or column over, or
end inside one; both sides of the rule's lines (2048 and 2^18 unknowns with
face coefficients, 3 2^17 with the constant operator, odd s); thin grids of
every orientation, whose bricks span one or two axes; the
moments kind with the stopping test in the first launch (to 131072 unknowns)
and without, the recurrence kind, no Jacobi, FP32+IR.  Two lockstep iterations
against the oracle (1e-10; 1e-4 for the FP32 Gram matrix), and, where the pairs
repeat the single steps' operations, the FP32 iterates against those bit for
bit."""
import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import make_operator, oracle_rhs, rel

pytestmark = pytest.mark.gpu

# (operator, dims, s, options, launches that form two columns)
CASES = [("faces", (16, 16, 8), 4, {}, 2), ("faces", (17, 9, 15), 6, {}, 3), ("faces", (16, 16, 7), 4, {}, 0),
         ("faces", (24, 23, 25), 5, {}, 0), ("faces", (13, 14, 15), 2, dict(precond=False), 1),
         ("faces", (64, 64, 64), 4, {}, 2), ("faces", (65, 64, 64), 4, {}, 0), ("faces", (50, 51, 52), 4, {}, 2),
         ("faces", (128, 9, 9), 4, dict(gram="recurrence"), 2), ("faces", (512, 2, 4), 4, {}, 2), ("faces", (1, 3000, 1), 4, {}, 2),
         ("const", (1, 1000, 500), 4, {}, 2), ("const", (500001, 1, 1), 5, {}, 2), ("const", (3, 3, 60000), 4, {}, 2),
         ("const", (900, 600, 1), 2, {}, 1), ("const", (2, 1, 1), 1, {}, 0), ("const", (1, 1, 3), 2, {}, 1),
         ("const", (17, 1030, 2), 3, dict(precond=False), 1),
         ("const", (8, 8, 8), 8, {}, 4), ("const", (5, 4, 3), 4, {}, 2), ("const", (9, 9, 9), 16, {}, 8),
         ("const", (31, 16, 33), 4, dict(precond=False), 2), ("const", (72, 73, 74), 4, {}, 2),
         ("const", (64, 96, 64), 4, {}, 2), ("const", (20, 21, 22), 6, dict(gram="apply"), 2)]


@pytest.mark.parametrize("op,dims,s,kw,pairs", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_bricks_fp64(hip, op, dims, s, kw, pairs):
    pr = (gen.small_faces3d if op == "faces" else gen.small_poisson3d)(*dims, seed=2, s=s, nu=20)
    A, b = oracle_rhs(pr)
    x = np.zeros(pr.n)
    precond = 1 if kw.get("precond", True) else 0
    lo, hi = (pr.lmin, pr.lmax) if precond else (0.0, 40.0 if op == "faces" else 12.0)
    with hip.Solver(make_operator(hip, pr, "stencil"), s, 20, lo, hi, max_outer=3, record_history=True, **kw) as sv:
        assert sv.basis_pairs == pairs
        rho = []
        for k in range(2):
            xt = torch.as_tensor(x, device="cuda:0")
            g = sv.step(torch.as_tensor(b, device="cuda:0"), xt)
            o = oracle.step(A, b, x, s, 20, lo, hi, precond=precond)
            rho.append(o["rnorm"])
            for key in ("G", "ctil", "atil"):
                assert rel(g[key], o[key]) <= 1e-10, (k, key)
            x = xt.cpu().numpy()
            assert rel(x, o["x"]) <= 1e-10, k
        got, st = sv.solve(torch.as_tensor(b, device="cuda:0"), None, 1e-14, raise_on_error=False, history=True)
        assert abs(st.hist_relres[1] - rho[1] / rho[0]) <= 1e-9 * rho[1] / rho[0]
        zero, st = sv.solve(torch.zeros(pr.n, dtype=torch.float64, device="cuda:0"), None, 1e-8)
        assert st.outer_iters == 0 and not zero.any()


@pytest.mark.parametrize("dims,s", [((8, 8, 8), 8), ((9, 17, 16), 4), ((33, 31, 20), 16), ((72, 73, 74), 4)])
def test_bricks_fp32(hip, dims, s):
    pr = gen.small_poisson3d(*dims, seed=3, s=s, nu=20)
    A, b = oracle_rhs(pr)
    bt = torch.as_tensor(b, device="cuda:0")
    out = []
    for steps in (0, 1):
        with hip.Solver(hip.Operator.stencil(*dims), s, 20, pr.lmin, pr.lmax, max_outer=2, precision="fp32ir",
                        gram="recurrence", autotune=False, basis_steps=steps) as sv:
            assert sv.basis_pairs == (0 if steps else s // 2)
            g = sv.step(bt, torch.zeros_like(bt))
            o = oracle.step(A, b, np.zeros(pr.n), s, 20, pr.lmin, pr.lmax)
            assert rel(g["G"], o["G"]) < 1e-4
            out.append(sv.solve(bt, None, 1e-15, raise_on_error=False)[0].cpu().numpy())
    assert np.array_equal(out[0], out[1])
