"""Small systems on the GPU at the lines of the short outer iteration: blocks of
one wave up to 32768 unknowns (a basis column per launch, or two in bricks), the
stopping test inside the first basis launch and the products' sums inside the Gram solve up to 131072.  Both sides of each
line, widths of few and many products, against the oracle: two lockstep
iterations (1e-10), the residual history of a solve, and the stops (limit of
iterations, zero and non-finite right-hand sides, an initial guess that is the
solution)."""
import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import make_operator, oracle_rhs, rel

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

CASES = [("faces", (32, 32, 32), 16), ("faces", (3, 10923, 1), 15), ("faces", (64, 64, 32), 31),
         ("faces", (3, 43691, 1), 16), ("csr", (32, 32, 32), 2), ("csr", (64, 64, 32), 16), ("27", (64, 64, 32), 8),
         ("27", (3, 43691, 1), 8), ("faces", (1, 1, 1), 1), ("csr", (13, 5, 1), 1)]


def t64(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)


@pytest.mark.parametrize("op,dims,s", CASES)
def test_lockstep_and_history(hip, op, dims, s):
    mk = gen.small_poisson27 if op == "27" else gen.small_faces3d
    pr = mk(*dims, seed=s, s=s, nu=20)
    A, b = oracle_rhs(pr)
    x = np.zeros(pr.n)
    with hip.Solver(make_operator(hip, pr, "csr" if op == "csr" else "stencil"), s, 20, pr.lmin, pr.lmax, max_outer=4,
                    record_history=True) as sv:
        assert sv.gram_kind == "moments"
        res = []
        for k in range(2 if pr.n > 1 else 1):
            xt = t64(x)
            g = sv.step(t64(b), xt)
            o = oracle.step(A, b, x, s, 20, pr.lmin, pr.lmax)
            res.append(o["rnorm"])
            assert abs(g["rnorm"] - o["rnorm"]) <= 1e-12 * o["rnorm"]
            for key in ("G", "ctil", "atil"):
                assert rel(g[key], o[key]) <= 1e-10, (k, key)
            x = xt.cpu().numpy()
            assert rel(x, o["x"]) <= 1e-10, k
        got, st = sv.solve(t64(b), None, 1e-9, raise_on_error=False, history=True)
        assert st.outer_iters <= 4 and abs(st.res0 - res[0]) <= 1e-12 * res[0]
        assert st.hist_relres[0] == 1.0 and st.hist_relres.size == st.outer_iters + 1
        if len(res) > 1:
            assert abs(st.hist_relres[1] - res[1] / res[0]) <= 1e-9 * res[1] / res[0]
        true = np.linalg.norm(b - oracle.spmv(A, got.cpu().numpy())) / np.linalg.norm(b)
        assert abs(st.rel_res - true) <= 1e-9 * true + 1e-15


@pytest.mark.parametrize("dims", [(9, 8, 7), (32, 32, 32), (40, 40, 41)])
def test_stops(hip, dims):
    pr = gen.small_faces3d(*dims, seed=1, s=8, nu=20)
    A, b = oracle_rhs(pr)
    op = make_operator(hip, pr, "stencil")
    with hip.Solver(op, 8, 20, pr.lmin, pr.lmax, max_outer=3) as sv:
        x, st = sv.solve(t64(b), None, 1e-14, raise_on_error=False)
        assert st.outer_iters == 3 and st.status == 5
        x, st = sv.solve(t64(0 * b), None, 1e-8)
        assert st.outer_iters == 0 and st.status == 0 and not x.any()
        bad = b.copy()
        bad[pr.n // 2] = np.nan
        x, st = sv.solve(t64(bad), None, 1e-8, raise_on_error=False)
        assert st.outer_iters == 0 and st.status == 6 and not x.any()
        again, st = sv.solve(t64(b), None, 1e-14, raise_on_error=False)  # the state of a stop does not stay
        assert st.outer_iters == 3
    with hip.Solver(op, 8, 20, pr.lmin, pr.lmax, max_outer=0) as sv:
        x, st = sv.solve(t64(b), None, 1e-8, raise_on_error=False)
        assert st.outer_iters == 0 and st.status == 5 and st.rel_res == 1.0


# blocks of one wave, of four, bricks of sixteen; the last of each also without the
# test in the launch
STARTS = [("csr", (9, 8, 7)), ("csr", (32, 32, 32)), ("csr", (40, 40, 41)), ("27", (40, 40, 41)), ("7", (9, 8, 7)),
          ("7", (40, 40, 41)), ("csr", (51, 52, 53)), ("7", (51, 52, 53))]


@pytest.mark.parametrize("op,dims", STARTS, ids=lambda v: str(v).replace(" ", ""))
def test_starts(hip, op, dims):
    """A start from the solution (integers on a constant operator: the residual
    is exactly zero) stops at once and stays as it is; from any other guess the
    first iterate is the oracle's from there (1e-10)."""
    pr = (gen.small_poisson27 if op == "27" else gen.small_poisson3d)(*dims, seed=5, s=8, nu=20)
    A, b = oracle_rhs(pr)
    r = gen.rng(12)
    whole = np.rint(50 * gen.uniform(r, pr.n))
    guess = gen.uniform(r, pr.n)
    o = oracle.step(A, b, guess, 8, 20, pr.lmin, pr.lmax)
    with hip.Solver(make_operator(hip, pr, "csr" if op == "csr" else "stencil"), 8, 20, pr.lmin, pr.lmax,
                    max_outer=1) as sv:
        for _ in range(3):  # a stop in the first launch, then a solve that goes on
            x, st = sv.solve(t64(oracle.spmv(A, whole)), t64(whole), 1e-8)
            assert (st.outer_iters, st.status, st.rel_res, st.res0) == (0, 0, 0.0, 0.0)
            assert np.array_equal(x.cpu().numpy(), whole)
            x, st = sv.solve(t64(b), t64(guess), 1e-14, raise_on_error=False)
            assert (st.outer_iters, st.status) == (1, 5)
            assert abs(st.res0 - o["rnorm"]) <= 1e-12 * o["rnorm"]
            assert rel(x.cpu().numpy(), o["x"]) <= 1e-10
