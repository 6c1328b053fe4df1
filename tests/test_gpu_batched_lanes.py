"""Two points per lane in the batched band kernels, where the lanes can go
wrong: rows of odd length (a lane's second point begins the next row, or the
first or last row of a band), rows of one and two points, a plane that fills a
block exactly or by all but one point, single planes.  One outer iteration and
two over the two-step basis equal the same over single steps bit for bit (the
same operations in the same order), FP64 and FP32; the moments kind is held to
the oracle's x at 1e-10 after two."""
import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import rel

pytestmark = pytest.mark.gpu

GRIDS = {
    "odd_bands": [(33, 63, 5), (101, 29, 7)],
    "narrow": [(1, 900, 4), (1, 1300, 3), (2, 701, 5)],
    "full_planes": [(1024, 1, 3), (1023, 1, 4), (31, 33, 6), (32, 32, 1)],
    "wide_odd": [(341, 5, 3), (255, 9, 2), (7, 5, 33)],
}


def batch(grids, nrhs, faces):
    r = gen.rng(5)
    out = []
    for dims in grids:
        n = int(np.prod(dims))
        k = gen.face_coefficients(r, *dims, 1.0) if faces else (None, None, None)
        b = np.stack([gen.uniform(r, n) for _ in range(nrhs)])
        out.append((dims, k, gen.gershgorin_jacobi_bounds(), b))
    return out


def run(hip, systems, nrhs, s, outer, **kw):
    ops = [hip.Operator.stencil(*d, *k) for d, k, _, _ in systems]
    with hip.BatchedSolver(ops, nrhs, s, 20, [q[2][0] for q in systems], [q[2][1] for q in systems], max_outer=outer,
                           autotune=False, **kw) as bs:
        x, st = bs.solve([torch.as_tensor(q[3].ravel(), device="cuda:0") for q in systems], None, 1e-15,
                         raise_on_error=False)
        pairs = bs.basis_pairs
    return [v.cpu().numpy().reshape(nrhs, -1) for v in x], st, pairs


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("faces,precond", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("precision", ["fp64", "fp32ir"])
def test_two_points_per_lane(hip, name, faces, precond, precision):
    nrhs, s = 2, 4
    systems = batch(GRIDS[name], nrhs, faces)
    for outer in (1, 2):
        two, st2, pairs = run(hip, systems, nrhs, s, outer, gram="recurrence", precision=precision, precond=precond)
        one, st1, none = run(hip, systems, nrhs, s, outer, gram="recurrence", precision=precision, precond=precond,
                             basis_steps=1)
        assert pairs == s // 2 and none == 0
        for q in range(len(systems)):
            assert np.array_equal(two[q], one[q]), (outer, systems[q][0], rel(two[q], one[q]))
        for u, v in zip(st2, st1):
            assert u.outer_iters == v.outer_iters == outer and abs(u.rel_res - v.rel_res) <= 1e-12 * v.rel_res
    if precision == "fp64":
        mom, _, _ = run(hip, systems, nrhs, s, 2, gram="moments", precond=precond)
        for q, (dims, k, (lo, hi), b) in enumerate(systems):
            A = oracle.assemble_stencil7(*dims, *k)
            for r in range(nrhs):
                x = np.zeros(b.shape[1])
                for _ in range(2):
                    x = oracle.step(A, b[r], x, s, 20, lo, hi, precond=1 if precond else 0)["x"]
                assert rel(mom[q][r], x) <= 1e-10, (dims, r)
