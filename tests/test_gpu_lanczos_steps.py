"""Lanczos passes on the GPU where their chunks, buffers and sections can go
wrong: sizes around one block and around 1024 blocks of 256 rows, step counts
through the rotation of the three vectors and up to the largest, and start
vectors far from unit scale.  alpha and beta against the oracle entry by entry
(1e-10, as the recurrence's other tests), the Ritz values against LAPACK's
eigenvalues of the returned tridiagonal matrix (64 eps of its norm)."""
import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import make_operator, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,form,steps,scale", [
    ((1, 1, 1), "stencil", 1, 1.0), ((5, 3, 17), "stencil", 2, 1.0), ((16, 16, 1), "csr", 3, 1.0),
    ((257, 1, 1), "stencil", 4, 1.0), ((32, 16, 1), "stencil", 5, 1e140), ((31, 33, 1), "csr", 7, 1e-140),
    ((64, 64, 64), "stencil", 4, 1.0), ((3, 87382, 1), "csr", 6, 1.0), ((37, 41, 43), "stencil", 64, 1.0)])
def test_lanczos_steps(hip, dims, form, steps, scale):
    pr = gen.small_faces3d(*dims, seed=9, sigma=1.0, s=4, nu=10)
    A = oracle.problem_csr(pr)
    u = gen.uniform(gen.rng(3), pr.n) * scale
    few = min(steps, 24)  # beyond, rounding has grown past the comparison
    ref = oracle.lanczos(A, u, few)
    with hip.Solver(make_operator(hip, pr, form), 4, 10, pr.lmin, pr.lmax) as sv:
        got = sv.lanczos(torch.as_tensor(u, device="cuda:0"), steps)
        part = sv.lanczos(torch.as_tensor(u, device="cuda:0"), few)
    assert part["m"] == ref["m"]
    for key in ("alpha", "beta"):
        ended = ref["beta"][ref["m"] - 1] <= 1e-13 * np.abs(ref["alpha"]).max()
        k = ref["m"] - (key == "beta" and ended)  # the beta that ends the recurrence is rounding: zero exactly
        assert rel(part[key][:k], ref[key][:k]) <= 1e-10, key
        assert np.array_equal(got[key][:k], part[key][:k])
    m = got["m"]
    al, be = np.asarray(got["alpha"][:m]), np.asarray(got["beta"][:m - 1])
    ev = np.linalg.eigvalsh(np.diag(al) + np.diag(be, 1) + np.diag(be, -1))
    assert np.max(np.abs(np.asarray(got["ritz"][:m]) - ev)) <= 64 * np.finfo(float).eps * np.abs(ev).max()


@pytest.mark.parametrize("op", ["7", "27", "csr"])
def test_a_multiple_of_a_unit_vector(hip, op):
    """From a whole multiple of a unit vector, without Jacobi, on a constant
    operator: every entry is a whole number or its quotient by the norm, which is
    a whole number again, so that alpha_0 is the diagonal entry and beta_1 the root
    of the number of neighbours, to the bit."""
    mk = gen.small_poisson27 if op == "27" else gen.small_poisson3d
    pr = mk(12, 11, 10, seed=3, s=4, nu=5)
    e = np.zeros(pr.n)
    e[5 + 12 * (5 + 11 * 5)] = 1.0
    with hip.Solver(make_operator(hip, pr, "csr" if op == "csr" else "stencil"), 4, 5, 0.0, 60.0, precond=False) as sv:
        for a in (1.0, 49.0, 98.0, 103.0, 107.0, 161.0, 3e9):
            r = sv.lanczos(torch.as_tensor(a * e, device="cuda:0"), 2)
            k = 26.0 if op == "27" else 6.0
            assert (r["alpha"][0], r["beta"][0]) == (k, np.sqrt(k)), a
