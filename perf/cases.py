"""Performance cases: the work a user of the library has it do, through its public entry points.

listed() names the cases, draw() gives others of the same families and ranges, prepare() makes what
a user's program holds before the call (operator, right-hand side, solver handle), run() is one call
and its outputs, work() is the least that call must move and compute, exact() is the same result from
plain torch in 64 bits.

A solve runs a fixed number of outer iterations (max_outer), as an inner solver of an outer method
does: the amount of work then does not depend on where the residual happens to cross a tolerance.
The differentiable solve runs to a tight tolerance instead, as training against it needs.
"""
import math

import numpy as np
import torch

import paper_2512_09642_amd as lib

DEV = "cuda:0"
TOL = 1e-8       # stopping tolerance of the solves
GRAD_TOL = 1e-12  # of the differentiable solve


# --------------------------------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------------------------------

def listed():
    return [
        # The smallest real system: 2D 5-point Poisson on 64 x 64 given as CSR.  Latency and launches.
        dict(name="csr2d_64", kind="solve", op="csr2d", nx=64, ny=64, nz=1, s=8, nu=20, outer=24),
        # A general sparse matrix without any grid behind it: random symmetric pattern, rows of very
        # different lengths, an odd number of rows.
        dict(name="csr_random_30k", kind="solve", op="csr_random", nx=30011, ny=1, nz=1, s=8, nu=20, outer=6),
        # An assembled 3D diffusion matrix (variable coefficients) on an odd, ragged grid, as CSR.
        dict(name="csr_faces_101", kind="solve", op="csr_faces", nx=101, ny=97, nz=103, s=16, nu=25, outer=6),
        # The headline workload: 224^3 Poisson, matrix-free, s = 16, nu = 25.
        dict(name="poisson7_224", kind="solve", op="poisson7", nx=224, ny=224, nz=224, s=16, nu=25, outer=8),
        # The mixed-precision solver (FP32 basis inside FP64 refinement) on a large ragged grid.
        dict(name="poisson7_ir_187", kind="solve", op="poisson7", nx=187, ny=173, nz=191, s=16, nu=20, outer=6,
             precision="fp32ir"),
        # Variable-coefficient diffusion at the size of the differentiable workload: its forward solve.
        dict(name="faces7_128", kind="solve", op="faces7", nx=128, ny=128, nz=128, s=16, nu=25, outer=8),
        # Learning coefficients through the solver: forward, adjoint and coefficient gradients.
        dict(name="grad_45", kind="grad", nx=45, ny=41, nz=47, s=16, nu=25),
        # The paper's operator and size: 27-point, 230^3, s = 20, nu = 30.
        dict(name="poisson27_230", kind="solve", op="poisson27", nx=230, ny=230, nz=230, s=20, nu=30, outer=4),
        # Spectrum bounds for the basis before a first solve: 10 Lanczos steps on 128^3 faces.
        dict(name="lanczos_128", kind="lanczos", nx=128, ny=128, nz=128, steps=10),
        # Serving many uneven systems at once: cubes of 32 to 96 a side, 8 right-hand sides each.
        dict(name="batched_20x8", kind="batched", nsys=20, lo=32, hi=96, nrhs=8, s=16, nu=25, outer=4),
        # A batch of small uneven systems in mixed precision: launches and a half-empty chip.
        dict(name="batched_ir_12x3", kind="batched", nsys=12, lo=9, hi=33, nrhs=3, s=8, nu=20, outer=6,
             precision="fp32ir"),
        # The coarse-grid solve of a two-level hierarchy, streamed, at the paper's size (n_c about 5000).
        dict(name="coarse_17", kind="coarse", nx=17, ny=17, nz=17, nu=20, formed=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, lo, hi):
    """Three sides around one log-uniform size, each its own by up to 10%."""
    m = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return [max(lo, min(hi, int(round(m * rng.uniform(0.9, 1.1))))) for _ in range(3)]


def draw(rng):
    family = rng.choice(["csr2d", "csr_random", "csr_faces", "poisson7", "poisson7_ir", "faces7", "grad",
                         "poisson27", "lanczos", "batched", "batched_ir", "coarse"])
    s, nu = rng.choice([8, 9, 10, 13, 16, 17, 20, 24]), rng.choice([15, 20, 25, 30])
    outer = rng.randint(2, 4)
    if family == "csr2d":
        return dict(kind="solve", op="csr2d", nx=_log(rng, 40, 300), ny=_log(rng, 40, 300), nz=1,
                    s=rng.choice([6, 8, 9, 12]), nu=nu, outer=rng.randint(4, 16))
    if family == "csr_random":
        return dict(kind="solve", op="csr_random", nx=_log(rng, 2000, 40000), ny=1, nz=1, s=rng.choice([6, 8, 9]),
                    nu=nu, outer=rng.randint(2, 5))
    if family in ("csr_faces", "faces7"):
        nx, ny, nz = _sides(rng, 20, 110 if family == "csr_faces" else 140)
        return dict(kind="solve", op=family, nx=nx, ny=ny, nz=nz, s=s, nu=nu, outer=outer)
    if family in ("poisson7", "poisson7_ir"):
        nx, ny, nz = _sides(rng, 24, 224)
        c = dict(kind="solve", op="poisson7", nx=nx, ny=ny, nz=nz, s=s, nu=nu, outer=outer)
        return dict(c, precision="fp32ir") if family == "poisson7_ir" else c
    if family == "grad":
        nx, ny, nz = _sides(rng, 12, 48)
        return dict(kind="grad", nx=nx, ny=ny, nz=nz, s=rng.choice([8, 12, 16]), nu=25)
    if family == "poisson27":
        nx, ny, nz = _sides(rng, 24, 200)
        return dict(kind="solve", op="poisson27", nx=nx, ny=ny, nz=nz, s=rng.choice([8, 10, 13, 20]), nu=nu,
                    outer=rng.randint(2, 3))
    if family == "lanczos":
        nx, ny, nz = _sides(rng, 24, 140)
        return dict(kind="lanczos", nx=nx, ny=ny, nz=nz, steps=rng.randint(5, 10))
    if family == "batched":
        return dict(kind="batched", nsys=rng.randint(4, 16), lo=rng.randint(12, 32), hi=rng.randint(48, 96),
                    nrhs=rng.randint(1, 8), s=rng.choice([8, 9, 16]), nu=nu, outer=outer)
    if family == "batched_ir":
        return dict(kind="batched", nsys=rng.randint(3, 12), lo=rng.randint(6, 12), hi=rng.randint(20, 40),
                    nrhs=rng.randint(1, 8), s=rng.choice([6, 8, 9]), nu=nu, outer=outer, precision="fp32ir")
    nx, ny, nz = _sides(rng, 5, 20)
    return dict(kind="coarse", nx=nx, ny=ny, nz=nz, nu=rng.choice([10, 20]), formed=rng.random() < 0.5)


# --------------------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(g, n):
    """n draws from U[-1, 1]."""
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * 2 - 1


def _faces(g, nx, ny, nz, sigma):
    """Log-normal face coefficients exp(sigma Z), boundary faces included."""
    return [torch.exp(sigma * torch.randn(n, generator=g, device=DEV, dtype=torch.float64))
            for n in ((nx + 1) * ny * nz, nx * (ny + 1) * nz, nx * ny * (nz + 1))]


def _poisson_bounds(sides):
    """Exact extreme eigenvalues of D^-1 A for constant-coefficient Poisson."""
    c = sum(math.cos(math.pi / (m + 1)) for m in sides) / len(sides)
    return 1.0 - c, 1.0 + c


def _poisson27_bounds(sides):
    c = [math.cos(math.pi / (m + 1)) for m in sides]
    p = [a * b * d for a in (1 - 2 * c[0], 1 + 2 * c[0]) for b in (1 - 2 * c[1], 1 + 2 * c[1])
         for d in (1 - 2 * c[2], 1 + 2 * c[2])]
    return (27.0 - max(p)) / 26.0, (27.0 - min(p)) / 26.0


def _grid_csr(nx, ny, nz, faces):
    """The 5- or 7-point operator of the faces (None: all 1) as CSR, columns ascending."""
    n = nx * ny * nz
    p = torch.arange(n, device=DEV)
    i, j, k = p % nx, (p // nx) % ny, p // (nx * ny)
    if faces is None:
        one = torch.ones(n, device=DEV, dtype=torch.float64)
        fw = fe = fs = fn = one
        fb = ft = one if nz > 1 else one * 0
    else:
        kx, ky, kz = (f.reshape(sh) for f, sh in zip(faces, ((nz, ny, nx + 1), (nz, ny + 1, nx), (nz + 1, ny, nx))))
        fw, fe = kx[:, :, :-1].reshape(-1), kx[:, :, 1:].reshape(-1)
        fs, fn = ky[:, :-1].reshape(-1), ky[:, 1:].reshape(-1)
        fb, ft = kz[:-1].reshape(-1), kz[1:].reshape(-1)
    diag = ((((fw + fe) + fs) + fn) + fb) + ft
    yes = torch.ones(n, device=DEV, dtype=torch.bool)
    cols = torch.stack([p - nx * ny, p - nx, p - 1, p, p + 1, p + nx, p + nx * ny], 1)
    vals = torch.stack([-fb, -fs, -fw, diag, -fe, -fn, -ft], 1)
    mask = torch.stack([k > 0, j > 0, i > 0, yes, i < nx - 1, j < ny - 1, k < nz - 1], 1)
    rp = torch.zeros(n + 1, device=DEV, dtype=torch.int64)
    rp[1:] = mask.sum(1).cumsum(0)
    return rp.to(torch.int32), cols[mask].to(torch.int32), vals[mask]


def _random_csr(g, n):
    """Random symmetric, strictly diagonally dominant matrix: each row draws 0 to 30 partners, the
    pattern is the union with its transpose, values U[-1, 1], diagonal 1 + sum of |row|."""
    k = torch.randint(0, 31, (n,), generator=g, device=DEV)
    a = torch.repeat_interleave(torch.arange(n, device=DEV), k)
    b = torch.randint(0, n, (int(a.numel()),), generator=g, device=DEV)
    a, b = a[a != b], b[a != b]
    pair = torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b))
    lo, hi = pair // n, pair % n
    v = _uniform(g, int(pair.numel()))
    diag = torch.ones(n, dtype=torch.float64)  # on the host: sums in a fixed order
    for end in (lo, hi):
        diag.index_add_(0, end.cpu(), v.abs().cpu())
    diag = diag.to(DEV)
    idx = torch.arange(n, device=DEV)
    key = torch.cat([lo * n + hi, hi * n + lo, idx * n + idx])
    val = torch.cat([v, v, diag])
    key, order = torch.sort(key)
    rp = torch.zeros(n + 1, device=DEV, dtype=torch.int64)
    rp[1:] = torch.bincount(key // n, minlength=n).cumsum(0)
    return rp.to(torch.int32), (key % n).to(torch.int32), val[order]


def _batch_sides(case):
    """Sides from lo to hi, evenly spread, in a mixed order that is the case's own."""
    m, lo, hi = case["nsys"], case["lo"], case["hi"]
    sides = [int(round(lo + (hi - lo) * q / max(1, m - 1))) for q in range(m)]
    return sides[::3] + sides[1::3] + sides[2::3]


def _problem(case, seed):
    """Operator data, bounds and right-hand side(s) of a case: what both prepare and exact start from."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "batched":
        sides = _batch_sides(case)
        faces = [_faces(g, m, m, m, 1.0) for m in sides]
        b = [_uniform(g, m ** 3 * case["nrhs"]) for m in sides]
        return dict(sides=sides, faces=faces, b=b, bounds=(0.0, 2.0))
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if kind == "coarse":
        return dict(faces=_faces(g, 2 * nx + 1, 2 * ny + 1, 2 * nz + 1, 1.0), f=_uniform(g, nx * ny * nz))
    op = case.get("op", "faces7")
    out = dict(n=nx * ny * nz, faces=None, csr=None, bounds=(0.0, 2.0))
    if op == "csr2d":
        out["csr"], out["bounds"] = _grid_csr(nx, ny, 1, None), _poisson_bounds((nx, ny))
    elif op == "csr_random":
        out["csr"] = _random_csr(g, nx)
    elif op == "csr_faces":
        out["csr"] = _grid_csr(nx, ny, nz, _faces(g, nx, ny, nz, 0.5))
    elif op == "faces7":
        out["faces"] = _faces(g, nx, ny, nz, 0.5)
    elif op == "poisson7":
        out["bounds"] = _poisson_bounds((nx, ny, nz))
    else:
        out["bounds"] = _poisson27_bounds((nx, ny, nz))
    out["b"] = _uniform(g, out["n"])
    if kind == "grad":
        out["target"] = _uniform(g, out["n"])
    return out


def _host(arrays):
    """Operators come from an assembly on the host."""
    return [a.cpu() for a in arrays]


def prepare(case, seed):
    kind, p = case["kind"], _problem(case, seed)
    if kind == "coarse":
        op = lib.Operator.stencil(*(2 * case[a] + 1 for a in ("nx", "ny", "nz")), *_host(p["faces"]))
        return dict(case=case, f=p["f"], solver=lib.CoarseSolver(op, formed=case["formed"]))
    precision = case.get("precision", "fp64")
    lo, hi = p["bounds"]
    if kind == "batched":
        ops = [lib.Operator.stencil(m, m, m, *_host(f)) for m, f in zip(p["sides"], p["faces"])]
        sv = lib.BatchedSolver(ops, case["nrhs"], case["s"], case["nu"], [lo] * len(ops), [hi] * len(ops),
                               precision=precision, max_outer=case["outer"])
        return dict(case=case, b=p["b"], solver=sv)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    if p["csr"] is not None:
        op = lib.Operator.csr(*_host(p["csr"]))
    elif case.get("op") == "poisson27":
        op = lib.Operator.stencil27(nx, ny, nz)
    elif p["faces"] is not None:
        op = lib.Operator.stencil(nx, ny, nz, *_host(p["faces"]))
    else:
        op = lib.Operator.stencil(nx, ny, nz)
    if kind == "lanczos":
        return dict(case=case, u=p["b"], solver=lib.Solver(op, 16, 25, lo, hi))
    if kind == "grad":
        return dict(case=case, coeffs=torch.cat(p["faces"]), b=p["b"], target=p["target"],
                    solver=lib.Solver(op, case["s"], case["nu"], lo, hi))
    # the FP32 Gram sums depend on the tuned schedule: a program that wants the same digits on every
    # machine turns the tuner off
    sv = lib.Solver(op, case["s"], case["nu"], lo, hi, precision=precision, max_outer=case["outer"],
                    autotune=precision == "fp64")
    return dict(case=case, b=p["b"], solver=sv)


# --------------------------------------------------------------------------------------------------
# one call
# --------------------------------------------------------------------------------------------------

def run(state):
    case, sv = state["case"], state["solver"]
    kind = case["kind"]
    if kind == "coarse":
        return dict(u=sv.fgs(state["f"], case["nu"]))
    if kind == "lanczos":
        r = sv.lanczos(state["u"], case["steps"])
        return dict(alpha=r["alpha"], beta=r["beta"], ritz=r["ritz"], m=r["m"])
    if kind == "batched":
        x, st = sv.solve(state["b"], None, TOL, raise_on_error=False)
        return dict(x=x, iters=np.array([v.outer_iters for v in st]), relres=np.array([v.rel_res for v in st]))
    if kind == "grad":
        k = state["coeffs"].detach().requires_grad_(True)
        b = state["b"].detach().requires_grad_(True)
        x = lib.sstep_solve(k, b, sv, GRAD_TOL)
        loss = 0.5 * (x - state["target"]).square().sum()
        loss.backward()
        return dict(x=x.detach(), dk=k.grad, db=b.grad)
    x, st = sv.solve(state["b"], None, TOL, raise_on_error=False)
    return dict(x=x, iters=st.outer_iters, relres=st.rel_res)


# --------------------------------------------------------------------------------------------------
# the least one call moves and computes
# --------------------------------------------------------------------------------------------------

def _solve_work(n, s, w, per_row_bytes, per_row_flops):
    """One outer iteration on n unknowns: b, x and the operator read, x written, every basis column
    written once and read once (the step lengths are known only after the last), s operator products
    and a residual, 2 s + 1 inner products and the update."""
    return (n * (8.0 * 3 + per_row_bytes + 2.0 * s * w), n * ((s + 1) * (per_row_flops + 6.0) + 2.0 * (3 * s + 1)))


def work(case):
    kind = case["kind"]
    if kind == "batched":
        w = 4 if case.get("precision") == "fp32ir" else 8
        bytes_ = flops = 0.0
        for m in _batch_sides(case):
            a, f = _solve_work(m ** 3, case["s"], w, 0, 18)
            bytes_ += case["outer"] * (case["nrhs"] * a + 24.0 * m ** 3)
            flops += case["outer"] * case["nrhs"] * f
        return dict(bytes=bytes_, flops=flops)
    n = case["nx"] * case["ny"] * case["nz"]
    if kind == "coarse":
        nf = (2 * case["nx"] + 1) * (2 * case["ny"] + 1) * (2 * case["nz"] + 1)
        return dict(bytes=8.0 * (3 * nf + 2 * n), flops=case["nu"] * n * (27 * 20.0 if not case["formed"] else 54.0))
    if kind == "lanczos":
        return dict(bytes=case["steps"] * 8.0 * n * (3 + 4), flops=case["steps"] * n * 26.0)
    if kind == "grad":
        # about as many outer iterations forward and backward as the grid is wide over two
        a, f = _solve_work(n, case["s"], 8, 24, 18)
        k = max(case["nx"], case["ny"], case["nz"])
        return dict(bytes=k * a + 8.0 * 8 * n, flops=k * f + 9.0 * n)
    w = 4 if case.get("precision") == "fp32ir" else 8
    per_row = {"csr2d": (60, 10), "csr_random": (12 * 31, 62), "csr_faces": (84, 14), "poisson7": (0, 7),
               "faces7": (24, 18), "poisson27": (0, 27)}[case["op"]]
    a, f = _solve_work(n, case["s"], w, *per_row)
    return dict(bytes=case["outer"] * a, flops=case["outer"] * f)


# --------------------------------------------------------------------------------------------------
# the same results in plain torch, 64 bits
# --------------------------------------------------------------------------------------------------

def _faces_apply(dims, faces):
    """u -> A u of the face operator on a grid, u of shape (..., n)."""
    nx, ny, nz = dims
    kx, ky, kz = (f.reshape(sh) for f, sh in zip(faces, ((nz, ny, nx + 1), (nz, ny + 1, nx), (nz + 1, ny, nx))))

    def apply(u):
        v = torch.nn.functional.pad(u.reshape(u.shape[:-1] + (nz, ny, nx)), (1, 1, 1, 1, 1, 1))
        c = v[..., 1:-1, 1:-1, 1:-1]
        y = kx[:, :, :-1] * (c - v[..., 1:-1, 1:-1, :-2]) + kx[:, :, 1:] * (c - v[..., 1:-1, 1:-1, 2:])
        y = y + ky[:, :-1] * (c - v[..., 1:-1, :-2, 1:-1]) + ky[:, 1:] * (c - v[..., 1:-1, 2:, 1:-1])
        y = y + kz[:-1] * (c - v[..., :-2, 1:-1, 1:-1]) + kz[1:] * (c - v[..., 2:, 1:-1, 1:-1])
        return y.reshape(u.shape)

    diag = kx[:, :, :-1] + kx[:, :, 1:] + ky[:, :-1] + ky[:, 1:] + kz[:-1] + kz[1:]
    return apply, diag.reshape(-1)


def _csr_apply(csr):
    rp, ci, v = csr
    n = rp.numel() - 1
    row = torch.repeat_interleave(torch.arange(n, device=DEV), (rp[1:] - rp[:-1]).to(torch.int64))
    ci = ci.to(torch.int64)
    diag = torch.zeros(n, device=DEV, dtype=torch.float64)
    diag[row[row == ci]] = v[row == ci]
    return (lambda u: torch.zeros_like(u).index_add_(-1, row, u.index_select(-1, ci) * v)), diag


def _box_apply(dims):
    """The 27-point operator: 27 u - (sum over the 3 x 3 x 3 box)."""
    nx, ny, nz = dims

    def apply(u):
        v = torch.nn.functional.pad(u.reshape(nz, ny, nx), (1, 1, 1, 1, 1, 1))
        v = v[:, :, :-2] + v[:, :, 1:-1] + v[:, :, 2:]
        v = v[:, :-2] + v[:, 1:-1] + v[:, 2:]
        v = v[:-2] + v[1:-1] + v[2:]
        return 27.0 * u - v.reshape(-1)

    return apply, torch.full((nx * ny * nz,), 26.0, device=DEV, dtype=torch.float64)


def _operator(case, p):
    dims = (case["nx"], case["ny"], case["nz"])
    if p["csr"] is not None:
        return _csr_apply(p["csr"])
    if case.get("op") == "poisson27":
        return _box_apply(dims)
    if p["faces"] is not None:
        return _faces_apply(dims, p["faces"])
    nx, ny, nz = dims
    ones = [torch.ones(m, device=DEV, dtype=torch.float64)
            for m in ((nx + 1) * ny * nz, nx * (ny + 1) * nz, nx * ny * (nz + 1))]
    return _faces_apply(dims, ones)


def _sstep(apply, diag, b, s, nu, lo, hi, outer, tol):
    """The s-step iteration written out: residual, Chebyshev basis, Gram system, nu forward
    Gauss-Seidel sweeps on the scaled system, update.  Returns x, iterations, relative residual."""
    theta, sigma = 2.0 / (hi - lo), (hi + lo) / 2.0
    x = torch.zeros_like(b)
    r0 = None
    for k in range(outer + 1):
        r = b - apply(x)
        rn = float(r.norm())
        r0 = rn if r0 is None else r0
        if rn < tol * r0 or k == outer:
            return x, k, rn / r0
        P, AP = [r / diag], []
        for j in range(s):
            AP.append(apply(P[j]))
            if j + 1 < s:
                t = theta * (AP[j] / diag - sigma * P[j])
                P.append(t if j == 0 else 2.0 * t - P[j - 1])
        P, AP = torch.stack(P), torch.stack(AP)
        G = (P @ AP.T).cpu().numpy()
        c = (P @ r).cpu().numpy()
        d = 1.0 / np.sqrt(np.diag(G))
        G, c = (d[:, None] * G) * d[None, :], d * c
        a = np.zeros(s)
        for _ in range(nu):
            for j in range(s):
                a[j] = c[j] - (G[j] @ a - G[j, j] * a[j])
        x = x + torch.as_tensor(d * a, device=DEV) @ P


def _exact_coarse(case, p):
    nc = (case["nx"], case["ny"], case["nz"])
    n = nc[0] * nc[1] * nc[2]
    if n > 9000:
        return None  # a dense coarse matrix: too slow here
    dims = tuple(2 * m + 1 for m in nc)
    apply, _ = _faces_apply(dims, p["faces"])

    def hat(m):
        h = torch.zeros(2 * m + 1, m, device=DEV, dtype=torch.float64)
        i = torch.arange(m, device=DEV)
        h[2 * i, i], h[2 * i + 1, i], h[2 * i + 2, i] = 0.5, 1.0, 0.5
        return h

    hx, hy, hz = (hat(m) for m in nc)
    A = torch.empty(n, n, device=DEV, dtype=torch.float64)
    idx = torch.arange(n, device=DEV)
    for q0 in range(0, n, 512):
        e = torch.zeros(min(512, n - q0), n, device=DEV, dtype=torch.float64)
        e[torch.arange(e.shape[0], device=DEV), idx[q0:q0 + e.shape[0]]] = 1.0
        v = e.reshape(-1, nc[2], nc[1], nc[0])
        v = v @ hx.T.contiguous()
        v = hy @ v
        v = (hz @ v.reshape(v.shape[0], nc[2], -1)).reshape(v.shape[0], -1)
        v = apply(v).reshape(-1, dims[2], dims[1], dims[0])
        v = v @ hx
        v = hy.T.contiguous() @ v
        A[q0:q0 + e.shape[0]] = (hz.T.contiguous() @ v.reshape(v.shape[0], dims[2], -1)).reshape(-1, n)
    u = torch.zeros(n, device=DEV, dtype=torch.float64)
    low, up = torch.tril(A), torch.triu(A, 1)
    for _ in range(case["nu"]):
        u = torch.linalg.solve_triangular(low, (p["f"] - up @ u)[:, None], upper=False)[:, 0]
    return dict(u=u)


def _exact_lanczos(case, p):
    apply, diag = _operator(case, p)
    m, u = case["steps"], p["b"]
    z, zp, beta = u / (diag * u * u).sum().sqrt(), None, 0.0
    al, be = [], []
    for _ in range(m):
        y = apply(z)
        al.append(float(z @ y))
        w = y / diag - al[-1] * z
        if zp is not None:
            w = w - beta * zp
        beta = float((diag * w * w).sum().sqrt())
        be.append(beta)
        z, zp = w / beta, z
    T = np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1)
    return dict(alpha=np.array(al), beta=np.array(be), ritz=np.linalg.eigvalsh(T), m=None)


def _cg(apply, diag, b):
    """Jacobi-preconditioned CG to the end of what 64 bits give."""
    x, r = torch.zeros_like(b), b.clone()
    z = r / diag
    d, rz, stop = z, float(r @ z), 1e-15 * float(b.norm())
    for _ in range(2000):
        q = apply(d)
        a = rz / float(d @ q)
        x, r = x + a * d, r - a * q
        if float(r.norm()) < stop:
            break
        z = r / diag
        rz, old = float(r @ z), rz
        d = z + (rz / old) * d
    return x


def _exact_grad(case, p):
    dims = (case["nx"], case["ny"], case["nz"])
    apply, diag = _faces_apply(dims, p["faces"])
    x = _cg(apply, diag, p["b"])
    lam = _cg(apply, diag, x - p["target"])
    nx, ny, nz = dims
    pad = torch.nn.functional.pad
    dk = []
    for axis, shape in ((0, (1, 1)), (1, (0, 0, 1, 1)), (2, (0, 0, 0, 0, 1, 1))):
        a, c = (pad(v.reshape(nz, ny, nx), shape) for v in (lam, x))
        dk.append(-(a.diff(dim=2 - axis) * c.diff(dim=2 - axis)).reshape(-1))
    return dict(x=x, dk=torch.cat(dk), db=lam)


def exact(case, seed):
    kind, p = case["kind"], _problem(case, seed)
    if kind == "coarse":
        return _exact_coarse(case, p)
    if kind == "lanczos":
        return _exact_lanczos(case, p)
    if kind == "grad":
        return _exact_grad(case, p)
    lo, hi = p["bounds"]
    if kind == "batched":
        xs, rr = [], []
        for m, faces, b in zip(p["sides"], p["faces"], p["b"]):
            apply, diag = _faces_apply((m, m, m), faces)
            got = [_sstep(apply, diag, v, case["s"], case["nu"], lo, hi, case["outer"], TOL)
                   for v in b.reshape(case["nrhs"], -1)]
            xs.append(torch.cat([v[0] for v in got]))
            rr += [v[2] for v in got]
        return dict(x=xs, iters=None, relres=np.array(rr))
    apply, diag = _operator(case, p)
    x, k, rr = _sstep(apply, diag, p["b"], case["s"], case["nu"], lo, hi, case["outer"], TOL)
    return dict(x=x, iters=k, relres=rr)
