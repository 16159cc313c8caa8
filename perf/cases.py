"""The work that programs have this library do, as cases that can be timed.

Three families of matrices, those of the benchmark and the tests:

* ``grid2d``, ``grid3d``: cell-centred finite-volume convection-diffusion on
  n^2 or n^3 cells of the unit square or cube (Dirichlet faces y = 0, 1,
  Neumann elsewhere), kappa log-uniform on blocks, first-order upwind;
* ``graph``: random geometric graph of n points with 6 to 14 neighbours a row,
  nonsymmetric, strictly diagonally dominant, points in no particular order.

Each case names one operation (``op``) and its sizes and options; see
``listed`` for what each stands for.  Inputs are made on the GPU, from the seed
alone, by the plain torch code below.
"""
from __future__ import annotations

import math

import torch

from paper_1105_3468_amd import Solver, autograd, gmg

DEV = "cuda"
F64 = torch.float64


# ------------------------------------------------------------------- cases
def listed():
    return [
        # one product with a small system matrix: what a program pays for the
        # smallest call there is
        dict(name="spmv_grid2d_64", op="spmv", family="grid2d", n=64, transposed=False),
        # one product with an unstructured matrix whose numbering has no locality
        dict(name="spmv_graph_500k", op="spmv", family="graph", n=500_000, transposed=False),
        # the preconditioner inside somebody else's Krylov method
        dict(name="apply_grid2d_1024", op="apply", family="grid2d", n=1024, contrast=4.0, velocity="rotating",
             tau=1e-6, adjoint=False),
        # its adjoint on a 3D grid
        dict(name="apply_adjoint_grid3d_128", op="apply", family="grid3d", n=128, contrast=6.0, velocity="const",
             tau=1e-5, adjoint=True),
        # a small solve, restarted: latency and launches count
        dict(name="solve_grid2d_64", op="solve", family="grid2d", n=64, contrast=3.0, velocity="const",
             tau=1e-4, restart=30, tol=1e-8, nrhs=1, fp32=False),
        # one million unknowns without restart, the library's default coarse
        # factors: a basis of up to 200 vectors, where the steps end
        dict(name="solve_grid2d_1024", op="solve", family="grid2d", n=1024, contrast=3.0, velocity="rotating",
             tau=1e-4, restart=200, tol=1e-8, nrhs=1, fp32=False),
        # two million unknowns in 3D to the gradients' tolerance: a basis of
        # over 400 vectors, at most 480 steps
        dict(name="solve_grid3d_128", op="solve", family="grid3d", n=128, contrast=5.0, velocity="const",
             tau=1e-4, restart=480, tol=1e-10, nrhs=1, fp32=False),
        # an unstructured solve with the FP32 preconditioner
        dict(name="solve_graph_500k_fp32", op="solve", family="graph", n=500_000, tau=1e-4, restart=30, tol=1e-8,
             nrhs=1, fp32=True),
        # one training step of the differentiable solve: assembly, setup, 16
        # right-hand sides forward and adjoint, gradients
        dict(name="grad_grid2d_512x16", op="grad", family="grid2d", n=512, contrast=3.0, velocity="const",
             tau=1e-6, restart=30, tol=1e-10, nrhs=16),
        # the same at the size of a quick experiment
        dict(name="grad_grid2d_32x16", op="grad", family="grid2d", n=32, contrast=3.0, velocity="const",
             tau=1e-6, restart=30, tol=1e-10, nrhs=16),
        # one training step through a general sparse matrix of odd size, few
        # right-hand sides
        dict(name="sparse_grad_graph_50k", op="sparse_grad", family="graph", n=50_021, tau=1e-4, restart=30,
             tol=1e-10, nrhs=3),
        # the finite-volume calls around a program's own solver: assembly and
        # the gradient for kappa
        dict(name="assemble_grid3d_128", op="assemble", family="grid3d", n=128, contrast=6.0, velocity="const", nrhs=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["spmv", "apply", "solve", "solve", "grad", "sparse_grad", "assemble"])
    grid = {"grid2d": dict(contrast=3.0, velocity=rng.choice(["const", "rotating"]), tau=rng.choice([1e-4, 1e-6])),
            "grid3d": dict(contrast=5.0, velocity="const", tau=rng.choice([1e-4, 1e-5])),
            "graph": dict(tau=1e-4)}
    if op == "spmv":
        f = rng.choice(["grid2d", "grid3d", "graph"])
        n = _log(rng, *{"grid2d": (32, 1024), "grid3d": (10, 128), "graph": (2_000, 500_000)}[f])
        return dict(op=op, family=f, n=n, transposed=rng.random() < 0.5)
    if op == "apply":
        f = rng.choice(["grid2d", "grid3d", "graph"])
        n = _log(rng, *{"grid2d": (32, 1024), "grid3d": (10, 96), "graph": (2_000, 500_000)}[f])
        return dict(op=op, family=f, n=n, adjoint=rng.random() < 0.5, **grid[f])
    if op == "solve":
        f = rng.choice(["grid2d", "grid3d", "graph"])
        n = _log(rng, *{"grid2d": (32, 512), "grid3d": (12, 64), "graph": (2_000, 300_000)}[f])
        fp32 = f != "grid3d" and rng.random() < 0.4
        return dict(op=op, family=f, n=n, restart=30 if f == "graph" else 200,
                    tol=1e-10 if fp32 and f == "grid2d" else 1e-8,
                    nrhs=rng.choice([1, 1, 2, 5, 16]) if f == "graph" else 1, fp32=fp32, **grid[f])
    if op == "grad":
        return dict(op=op, family="grid2d", n=_log(rng, 16, 256), contrast=3.0, velocity="const", tau=1e-6,
                    restart=30, tol=1e-10, nrhs=rng.choice([1, 2, 3, 7, 16]))
    if op == "sparse_grad":
        return dict(op=op, family="graph", n=_log(rng, 2_000, 100_000), tau=1e-4, restart=30, tol=1e-10,
                    nrhs=rng.choice([1, 2, 3, 8]))
    f = rng.choice(["grid2d", "grid3d"])
    return dict(op=op, family=f, n=_log(rng, *((32, 1500) if f == "grid2d" else (10, 128))), contrast=3.0,
                velocity="const", nrhs=rng.choice([1, 2, 5, 16]) if f == "grid2d" else rng.choice([1, 2, 3]))


# ------------------------------------------------------------------ inputs
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 8 + salt)
    return g


def _uniform(shape, g, lo=-1.0, hi=1.0):
    return lo + (hi - lo) * torch.rand(shape, generator=g, device=DEV, dtype=F64)


def _kappa(case, seed):
    """kappa per cell, x fastest: log-uniform on blocks (of 8 cells a side in
    3D, of 16 cells with the rotating velocity, else eight blocks a side)."""
    n, dim, c = case["n"], _dim(case), case.get("contrast", 3.0)
    blocks = max(1, n // 8) if dim == 3 else max(1, n // 16) if case.get("velocity") == "rotating" else 8
    kb = 10.0 ** _uniform((blocks,) * dim, _gen(seed, 1), -c, c)
    at = torch.arange(n, device=DEV) * blocks // n
    return (kb[at][:, at] if dim == 2 else kb[at][:, at][:, :, at]).reshape(-1).contiguous()


def _dim(case):
    return 3 if case["family"] == "grid3d" else 2


def _velocity(case):
    """Face velocities (x, y[, z]); face array d has n + 1 entries along d."""
    n, dim = case["n"], _dim(case)
    if case.get("velocity") == "rotating":
        t = torch.arange(n + 1, device=DEV, dtype=F64) / n
        psi = (10.0 / math.pi) * torch.sin(math.pi * t)[None, :] * torch.sin(math.pi * t)[:, None]
        return [((psi[1:, :] - psi[:-1, :]) * n).contiguous(), (-(psi[:, 1:] - psi[:, :-1]) * n).contiguous()]
    a = (1.0, 0.5) if dim == 2 else (1.0, 1.0, 1.0)
    return [torch.full([n + (dim - 1 - d == k) for k in range(dim)], a[d], device=DEV, dtype=F64) for d in range(dim)]


def _bands(n, dim, kap, vel):
    """{offset: (values, mask)} of the finite-volume matrix, differentiable in kap."""
    k, sh, h = kap.reshape((n,) * dim), (n,) * dim, 1.0 / n
    diag, out = torch.zeros(sh, device=kap.device, dtype=F64), {}
    for d in range(dim):
        ax = dim - 1 - d
        ka, kb = k.narrow(ax, 0, n - 1), k.narrow(ax, 1, n - 1)
        T = 2.0 * ka * kb / ((ka + kb) * h * h)
        F = vel[d].reshape([n + (ax == i) for i in range(dim)])
        hi, lo = F.narrow(ax, 1, n), -F.narrow(ax, 0, n)
        edge = torch.zeros_like(k.narrow(ax, 0, 1))
        one = torch.ones_like(T, dtype=torch.bool)
        no = torch.zeros_like(edge, dtype=torch.bool)
        below, above = torch.cat([edge, T], ax), torch.cat([T, edge], ax)
        diag = diag + below + above + hi.clamp(min=0) / h + lo.clamp(min=0) / h
        out[n ** d] = (hi.clamp(max=0) / h - above, torch.cat([one, no], ax))
        out[-(n ** d)] = (lo.clamp(max=0) / h - below, torch.cat([no, one], ax))
        if d == 1:
            walls = torch.zeros(n, device=kap.device, dtype=F64)
            walls[0] += 2.0 / (h * h)
            walls[-1] += 2.0 / (h * h)
            diag = diag + k * walls.reshape([n if i == ax else 1 for i in range(dim)])
    out[0] = (diag, torch.ones(sh, device=kap.device, dtype=torch.bool))
    return {o: (v.reshape(-1), m.reshape(-1)) for o, (v, m) in out.items()}


def _csr_of_bands(N, bands):
    offs = sorted(bands)
    mask = torch.stack([bands[o][1] for o in offs], 1)
    vals = torch.stack([bands[o][0] for o in offs], 1)
    cols = torch.arange(N, device=mask.device)[:, None] + torch.tensor(offs, device=mask.device)[None, :]
    rp = torch.zeros(N + 1, dtype=torch.int32, device=mask.device)
    rp[1:] = torch.cumsum(mask.sum(1), 0)
    return rp, cols[mask].to(torch.int32), vals[mask]


def _graph(n, seed):
    """Random geometric graph: per row 6 to 14 of the nearest points among the
    nine cells around it, off-diagonals -U(0.1, 1) with 10% asymmetry, diagonal
    1.05 times the row's sum of magnitudes."""
    g = _gen(seed, 2)
    pts = torch.rand((n, 2), generator=g, device=DEV, dtype=torch.float32)
    side = max(3, int(math.sqrt(n / 9.0)))
    cx = (pts * side).long().clamp(max=side - 1)
    cell = cx[:, 1] * side + cx[:, 0]
    order = torch.argsort(cell, stable=True)
    count = torch.bincount(cell, minlength=side * side)
    start = torch.cumsum(count, 0) - count
    cap = int(count.max())
    slot = torch.full((side * side + 1, cap), -1, dtype=torch.long, device=DEV)
    slot[cell[order], torch.arange(n, device=DEV) - start[cell[order]]] = order
    near = []
    for at in torch.arange(n, device=DEV).split(50_000):
        around = []
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                x, y = cx[at, 0] + dx, cx[at, 1] + dy
                ok = (x >= 0) & (x < side) & (y >= 0) & (y < side)
                around.append(slot[torch.where(ok, y * side + x, torch.full_like(x, side * side))])
        cand = torch.cat(around, 1)
        d = (pts[cand.clamp(min=0)] - pts[at][:, None, :]).square().sum(2)
        d = d.masked_fill((cand < 0) | (cand == at[:, None]), float("inf"))
        best, pick = torch.topk(d, 14, dim=1, largest=False)
        near.append(torch.where(torch.isinf(best), torch.full_like(pick, -1), torch.gather(cand, 1, pick)))
    near = torch.cat(near)
    k = (6 + torch.arange(n, device=DEV) % 9)[torch.randperm(n, generator=g, device=DEV)]  # the same entries for every seed
    keep = (near >= 0) & (torch.arange(14, device=DEV)[None, :] < k[:, None])
    rows = torch.arange(n, device=DEV)[:, None].expand(-1, 14)[keep]
    cols = near[keep]
    # one magnitude for each unordered pair: a hash of its two ends
    lo, hi = torch.minimum(rows, cols), torch.maximum(rows, cols)
    m = 0.1 + 0.9 * ((lo * 2654435761 + hi * 40503 + seed * 97) % 1000003).to(F64) / 1000003
    off = -m * (1.0 + 0.1 * _uniform(rows.shape, g))
    dsum = torch.zeros(n, device=DEV, dtype=F64).index_add_(0, rows, off.abs().clamp(min=0.01))
    rows, cols = torch.cat([rows, torch.arange(n, device=DEV)]), torch.cat([cols, torch.arange(n, device=DEV)])
    vals = torch.cat([off, 1.05 * dsum])
    key = torch.argsort(rows * n + cols)
    rp = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return rp, cols[key].to(torch.int32), vals[key]


def _matrix(case, seed):
    if case["family"] == "graph":
        return _graph(case["n"], seed)
    n, dim = case["n"], _dim(case)
    return _csr_of_bands(n ** dim, _bands(n, dim, _kappa(case, seed), _velocity(case)))


def _size(case):
    return case["n"] if case["family"] == "graph" else case["n"] ** _dim(case)


def _rhs(case, seed, salt):
    nrhs = case.get("nrhs", 1)
    return _uniform((_size(case),) if nrhs == 1 else (_size(case), nrhs), _gen(seed, salt))


def _maxit(case):
    return 600 if case["restart"] == 30 else case["restart"]


def _options(case):
    return dict(cf=4.0, ilut_tau=case["tau"], restart=case["restart"], maxit=_maxit(case))


def prepare(case, seed):
    op = case["op"]
    s = dict(case=case, op=op)
    if op in ("spmv", "apply", "solve"):
        # the handle that such a program sets up once per matrix
        s["solver"] = Solver(*_matrix(case, seed), cf=4.0, ilut_tau=case.get("tau", 1e-4))
        s["b"] = _rhs(case, seed, 3)
        return s
    if op == "sparse_grad":
        s["A"] = _matrix(case, seed)
    else:
        s["kappa"], s["vel"] = _kappa(case, seed), _velocity(case)
    s["b"], s["target"] = _rhs(case, seed, 3), _rhs(case, seed, 4)
    return s


# -------------------------------------------------------------------- pass
def run(s):
    case, op = s["case"], s["op"]
    if op == "spmv":
        return s["solver"].spmv(s["b"], transposed=case["transposed"])
    if op == "apply":
        return s["solver"].apply(s["b"], adjoint=case["adjoint"])
    if op == "solve":
        x, _ = s["solver"].solve(s["b"], tol=case["tol"], restart=case["restart"], maxit=_maxit(case),
                                 precond_fp32=int(case["fp32"]))
        return x
    if op == "grad":
        kap, b = s["kappa"].detach().requires_grad_(), s["b"].detach().requires_grad_()
        x = autograd.fv_solve(kap, b, case["n"], _dim(case), s["vel"], tol=case["tol"], **_options(case))
        (x - s["target"]).square().sum().backward()
        return dict(x=x.detach(), kappa_grad=kap.grad, b_grad=b.grad)
    if op == "sparse_grad":
        rp, ci, va = s["A"]
        va, b = va.detach().requires_grad_(), s["b"].detach().requires_grad_()
        x = autograd.sparse_solve(rp, ci, va, b, tol=case["tol"], **_options(case))
        (x - s["target"]).square().sum().backward()
        return dict(x=x.detach(), value_grad=va.grad, b_grad=b.grad)
    n, dim = case["n"], _dim(case)
    rp, ci, va = gmg.fv_assemble(n, dim, s["kappa"], s["vel"])
    return dict(rowptr=rp, col=ci, val=va, kappa_grad=gmg.fv_kappa_grad(n, dim, s["kappa"], s["b"], s["target"]))


# -------------------------------------------------------------------- work
def _entries(case):
    n = case["n"]
    return 11 * n if case["family"] == "graph" else 5 * n * n - 4 * n if _dim(case) == 2 else 7 * n ** 3 - 6 * n * n


def _steps(case):
    """FGMRES steps of one solve, about (35 and 170 at 64^2 and 1024^2 with the
    default coarse factors, 430 at 128^3; 14 on the graphs, whatever their
    size)."""
    digits = -math.log10(case["tol"]) / 8.0
    at = 14.0 if case["family"] == "graph" else 5.3 * case["n"] ** 0.5 if _dim(case) == 2 else 2.7 * case["n"] + 4
    if _dim(case) == 2 and case["tau"] < 1e-5:
        at *= 0.5
    return min(at * digits, _maxit(case))


def work(case):
    """Bytes and operations that a pass cannot do without.  A product reads the
    matrix (12 bytes an entry) and the vector and writes the result; the
    preconditioner reads A, its ILU(0) values and the coarse factors (about 6,
    20 and 3 entries an unknown on the 2D and 3D grids and the graphs) once;
    an FGMRES step takes one of each and two reads of the basis (against which
    it projects, then updates), writing its two new vectors."""
    N, nnz, op = _size(case), _entries(case), case["op"]
    if op == "spmv":
        return dict(bytes=12 * nnz + 20 * N, flops=2 * nnz)
    if op == "assemble":
        return dict(bytes=12 * nnz + 4 * N + 8 * N + 8 * _dim(case) * N + 8 * N + 16 * N * case["nrhs"] + 8 * N,
                    flops=40 * N + 16 * N * case["nrhs"])
    fill = {"graph": 3, "grid2d": 6, "grid3d": 20}[case["family"]] * N
    val = 4 if case.get("fp32") else 8
    cycle = dict(bytes=(4 + val) * (nnz + fill) + val * nnz + 16 * N, flops=4 * nnz + 2 * fill)
    if op == "apply":
        return cycle
    steps = _steps(case) * (1 if op == "solve" else 2)
    depth = min(_steps(case), case["restart"]) / 2
    cols = case["nrhs"]
    vecs = (16 * depth + 40) * N
    return dict(bytes=steps * (cycle["bytes"] + 12 * nnz + vecs * cols),
                flops=steps * cols * (cycle["flops"] + 2 * nnz + 8 * depth * N))


# ------------------------------------------------------------- exact values
def _product(rp, ci, va, x, transposed=False):
    rows = torch.repeat_interleave(torch.arange(rp.numel() - 1, device=DEV), (rp[1:] - rp[:-1]).long())
    i, j = (ci.long(), rows) if transposed else (rows, ci.long())
    v = va if x.dim() == 1 else va[:, None]
    return torch.zeros_like(x).index_add_(0, i, v * x[j])


def _exact_solve(case, A, b, transposed=False):
    """Dense elimination for small grids, Jacobi iteration for the strictly
    diagonally dominant graphs (its error falls by 1/1.05 a step); else None."""
    rp, ci, va = A
    N = rp.numel() - 1
    if case["family"] == "graph":
        rows = torch.repeat_interleave(torch.arange(N, device=DEV), (rp[1:] - rp[:-1]).long())
        d = va[rows == ci]
        d = d if b.dim() == 1 else d[:, None]
        x = torch.zeros_like(b)
        for _ in range(900):
            x = x + (b - _product(rp, ci, va, x, transposed)) / d
        return x
    if N > 4096:
        return None
    M = torch.sparse_csr_tensor(rp.long().cpu(), ci.long().cpu(), va.cpu(), (N, N)).to_dense()
    x = torch.linalg.solve(M.T if transposed else M, b.cpu().reshape(N, -1))
    return x.reshape(b.shape).to(DEV)


def _kappa_gradient(case, kap, vel, lam, x):
    """-sum_r lam_r^T (dA/dkappa) x_r by differentiating the assembled product."""
    n, dim = case["n"], _dim(case)
    kap = kap.detach().requires_grad_()
    lam, x = lam.reshape(kap.numel(), -1), x.reshape(kap.numel(), -1)
    at, total = torch.arange(kap.numel(), device=DEV), 0.0
    for o, (v, m) in _bands(n, dim, kap, vel).items():
        total = total - (v[m] * (lam[at[m]] * x[at[m] + o]).sum(1)).sum()
    return torch.autograd.grad(total, kap)[0]


def exact(case, seed):
    op = case["op"]
    if op == "apply":  # depends on the aggregates and the factors' drops
        return None
    if op == "assemble":
        kap, vel = _kappa(case, seed), _velocity(case)
        rp, ci, va = _matrix(case, seed)
        return dict(rowptr=rp, col=ci, val=va,
                    kappa_grad=_kappa_gradient(case, kap, vel, _rhs(case, seed, 3), _rhs(case, seed, 4)))
    if case["family"] != "graph" and op != "spmv" and _size(case) > 4096:
        return None
    A, b = _matrix(case, seed), _rhs(case, seed, 3)
    if op == "spmv":
        return _product(*A, b, case["transposed"])
    x = _exact_solve(case, A, b)
    if op == "solve":
        return x
    lam = _exact_solve(case, A, 2.0 * (x - _rhs(case, seed, 4)), transposed=True)
    if op == "grad":
        return dict(x=x, kappa_grad=_kappa_gradient(case, _kappa(case, seed), _velocity(case), lam, x), b_grad=lam)
    rows = torch.repeat_interleave(torch.arange(_size(case), device=DEV), (A[0][1:] - A[0][:-1]).long())
    return dict(x=x, value_grad=-(lam.reshape(b.shape[0], -1)[rows] * x.reshape(b.shape[0], -1)[A[1].long()]).sum(1),
                b_grad=lam)
