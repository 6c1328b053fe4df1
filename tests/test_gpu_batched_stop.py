"""Stopping test of a batch between residual and basis, on every path that
feeds it partials (band table with and without the moments kind, chunk tiles)
and at counts of pairs around the waves of a block.  Pairs stop at different
iterations, at once (zero right-hand side, exact initial guess), on a
non-finite norm and at the limit, beside pairs that go on; each ends where the
same system alone does: the same iteration count and status, x within 1e-9."""
import numpy as np
import pytest
import torch

import gen
from helpers import rel

pytestmark = pytest.mark.gpu


def t64(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


@pytest.mark.parametrize("kw", [dict(gram="moments"), dict(gram="recurrence"), dict(gram="recurrence", basis_steps=1),
                                dict(gram="stored")], ids=lambda k: "-".join(str(v) for v in k.values()))
@pytest.mark.parametrize("dims,nrhs", [([(12, 11, 10)], 1), ([(9, 8, 7), (20, 19, 18)], 2),
                                       ([(9, 8, 7), (40, 39, 4), (5, 5, 5)], 3)])
def test_pairs_stop_as_alone(hip, kw, dims, nrhs):
    r = gen.rng(11)
    s, nu, tol = 8, 20, 1e-9
    lo, hi = gen.gershgorin_jacobi_bounds()
    ops, bs_, xs = [], [], []
    for q, d in enumerate(dims):
        n = int(np.prod(d))
        ops.append(hip.Operator.stencil(*d, *gen.face_coefficients(r, *d, 1.0)))
        b = np.stack([gen.uniform(r, n) for _ in range(nrhs)])
        if nrhs > 1 and q == 0:
            b[1] = 0.0
        if nrhs > 2 and q == 1:
            b[0, n // 3] = np.inf
        bs_.append(b)
        xs.append(np.zeros_like(b))
    alone = [[] for _ in dims]
    for q in range(len(dims)):
        with hip.BatchedSolver([ops[q]], 1, s, nu, [lo], [hi], max_outer=6, **kw) as one:
            for k in range(nrhs):
                x, st = one.solve([t64(bs_[q][k])], [t64(xs[q][k])], tol, raise_on_error=False)
                alone[q].append((x[0].cpu().numpy(), st[0]))
    with hip.BatchedSolver(ops, nrhs, s, nu, [lo] * len(ops), [hi] * len(ops), max_outer=6, **kw) as bt:
        for _ in range(2):  # the state of a stop does not stay
            x, st = bt.solve([t64(b.ravel()) for b in bs_], [t64(v.ravel()) for v in xs], tol, raise_on_error=False)
            for q in range(len(dims)):
                got = x[q].cpu().numpy().reshape(nrhs, -1)
                for k in range(nrhs):
                    xa, sa = alone[q][k]
                    sb = st[q * nrhs + k]
                    assert (sb.outer_iters, sb.status) == (sa.outer_iters, sa.status), (q, k)
                    if sa.status != 6:
                        assert rel(got[k], xa) <= 1e-9 if np.any(xa) else not np.any(got[k]), (q, k)
                        assert abs(sb.rel_res - sa.rel_res) <= 1e-6 * sa.rel_res + 1e-14


@pytest.mark.parametrize("kw", [dict(gram="moments"), dict(gram="recurrence", basis_steps=1), dict(gram="stored"),
                                dict(precision="fp32ir")], ids=lambda k: "-".join(str(v) for v in k.values()))
def test_pairs_that_start_at_the_solution(hip, kw):
    """The first pair of every system starts at its solution (integers on the
    constant operator: the residual is exactly zero), stops at once and stays as it
    is; the others iterate from their own guess and end as from there alone."""
    r = gen.rng(13)
    dims, nrhs, s, tol = [(9, 8, 7), (40, 39, 4), (5, 5, 5)], 3, 8, 1e-9
    ops = [hip.Operator.stencil(*d) for d in dims]
    bounds = [gen.jacobi_poisson_bounds(*d) for d in dims]
    lo, hi = [v[0] for v in bounds], [v[1] for v in bounds]
    b, x0 = [], []
    for q, d in enumerate(dims):
        n = int(np.prod(d))
        x0.append(np.stack([np.rint(50 * gen.uniform(r, n))] + [gen.uniform(r, n) for _ in range(nrhs - 1)]))
        b.append(np.stack([gen.uniform(r, n) for _ in range(nrhs)]))
        with hip.Solver(ops[q], 1, 1, lo[q], hi[q]) as sv:
            b[q][0] = sv.apply(t64(x0[q][0])).cpu().numpy()
    with hip.BatchedSolver(ops, nrhs, s, 20, lo, hi, max_outer=2, **kw) as bt:
        for _ in range(2):
            x, st = bt.solve([t64(v.ravel()) for v in b], [t64(v.ravel()) for v in x0], tol, raise_on_error=False)
            for q in range(len(dims)):
                first = st[q * nrhs]
                assert (first.outer_iters, first.status, first.rel_res, first.res0) == (0, 0, 0.0, 0.0)
                assert np.array_equal(x[q].cpu().numpy().reshape(nrhs, -1)[0], x0[q][0])
    for q in range(len(dims)):
        with hip.BatchedSolver([ops[q]], 1, s, 20, lo[q:q + 1], hi[q:q + 1], max_outer=2, **kw) as one:
            for k in range(1, nrhs):
                xa, sa = one.solve([t64(b[q][k])], [t64(x0[q][k])], tol, raise_on_error=False)
                sb = st[q * nrhs + k]
                assert (sb.outer_iters, sb.status) == (sa[0].outer_iters, sa[0].status), (q, k)
                bar = 1e-5 if "precision" in kw else 1e-9
                assert rel(x[q].cpu().numpy().reshape(nrhs, -1)[k], xa[0].cpu().numpy()) <= bar, (q, k)
