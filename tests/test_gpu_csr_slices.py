"""The sliced form of CSR operators on the GPU: slices of 64 rows kept by their
offsets (column - row) or listed with their columns, in one matrix.

The matrix is block diagonal: a 27-point grid (27 offsets, several groups of
8), a random pattern (listed), a diagonal part (one offset), 5-point and
7-point grids; the parts do not end on slices, so slices straddle them, and
the last one is partial.  Products entry by entry against the oracle (the
rounding bound of a row's sum), non-finite entries reaching exactly the rows
that reference them, lockstep (1e-10) and new values on the same pattern."""
import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import rel

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def t64(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device=DEV)


def random_part(n, seed):
    r = np.random.default_rng(seed)
    k = 9 * n
    i, j = r.integers(0, n, k), r.integers(0, n, k)
    pair = np.unique(np.minimum(i, j)[i != j] * n + np.maximum(i, j)[i != j])
    lo, hi, v = pair // n, pair % n, r.uniform(-1, 1, pair.size)
    d = np.ones(n)
    np.add.at(d, lo, np.abs(v))
    np.add.at(d, hi, np.abs(v))
    R, C = np.concatenate([lo, hi, np.arange(n)]), np.concatenate([hi, lo, np.arange(n)])
    V = np.concatenate([v, v, d])
    o = np.lexsort((C, R))
    rp = np.concatenate([[0], np.cumsum(np.bincount(R, minlength=n))])
    return rp, C[o], V[o]


def block_diagonal(parts):
    rp, ci, v, n = [np.zeros(1, np.int64)], [], [], 0
    for p, c, x in parts:
        rp.append(np.asarray(p[1:], np.int64) + rp[-1][-1])
        ci.append(np.asarray(c, np.int64) + n)
        v.append(x)
        n += len(p) - 1
    return np.concatenate(rp).astype(np.int32), np.concatenate(ci).astype(np.int32), np.concatenate(v)


def matrix(kind):
    r = np.random.default_rng(5)
    if kind == "mixed":
        diag = (np.arange(201), np.arange(200), r.uniform(1, 2, 200))
        return block_diagonal([gen.poisson27_csr(9, 8, 7), random_part(333, 1), diag, gen.poisson2d_csr(23, 31),
                               gen.faces3d_csr(13, 11, 10, *gen.face_coefficients(gen.rng(3), 13, 11, 10, 0.5))])
    if kind == "one":
        return np.array([0, 1], np.int32), np.array([0], np.int32), np.array([3.0])
    if kind == "over_wave_blocks":  # above 32768 rows: blocks of four waves
        return block_diagonal([gen.poisson2d_csr(190, 173), random_part(700, 2)])
    return gen.poisson2d_csr(13, 5)  # 65 rows: one full slice and one of a single row


@pytest.mark.parametrize("kind", ["mixed", "one", "over_wave_blocks", "65_rows"])
def test_products_steps_and_new_values(hip, kind):
    rp, ci, v = matrix(kind)
    n = rp.size - 1
    x = np.random.default_rng(2).uniform(-1, 1, n)
    rows = np.repeat(np.arange(n), np.diff(rp))
    with hip.Solver(hip.Operator.csr(rp, ci, v), 4, 10, 0.0, 2.0) as sv:
        for scale in (1.0, 1.75):
            A = (rp, ci, scale * v)
            y = sv.apply(t64(x)).cpu().numpy()
            bound = np.zeros(n)
            np.add.at(bound, rows, np.abs(A[2] * x[ci]))
            assert np.all(np.abs(y - oracle.spmv(A, x)) <= (np.diff(rp) + 1) * 2.0 ** -52 * bound)
            bad = x.copy()
            bad[[0, n // 2, n - 1]] = np.nan, np.inf, np.nan
            hit = np.zeros(n, bool)
            hit[rows[~np.isfinite(bad[ci])]] = True
            assert np.array_equal(~np.isfinite(sv.apply(t64(bad)).cpu().numpy()), hit)
            if n > 4:
                g = t64(np.zeros(n))
                sv.step(t64(x), g)
                o = oracle.step(A, x, np.zeros(n), 4, 10, 0.0, 2.0)
                assert rel(g.cpu().numpy(), o["x"]) <= 1e-10
            sv.update_coefficients(hip.Operator.csr(rp, ci, 1.75 * v))
