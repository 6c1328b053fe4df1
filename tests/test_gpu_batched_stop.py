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
