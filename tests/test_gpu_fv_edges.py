"""Finite-volume assembly and its gradients where the kernels' tiles end:
row counts around multiples of the 256-row workgroups, one-cell grids, and
right-hand side counts around the powers of two that choose the lanes per
cell.  Assembly is bit-exact against the host generator; the gradients are
compared with extended-precision sums of the same terms, within 64 rounding
errors of the terms' magnitudes."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import autograd as AG  # noqa: E402
from paper_1105_3468_amd import gmg as G  # noqa: E402

EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("n,dim", [(1, 2), (2, 2), (15, 2), (16, 2), (17, 2), (33, 2), (1, 3), (2, 3), (6, 3), (8, 3),
                                   (13, 3)])
def test_assembly_at_tile_edges(n, dim):
    rng = np.random.default_rng(n + 100 * dim)
    kap = 10.0 ** rng.uniform(-3, 3, n ** dim)
    vel = W.velocity_rotating(10.0) if dim == 2 else W.velocity_const((1.0, -2.0, 0.5))
    rp, ci, va = W.fv_matrix(n, dim, kap, vel)
    got = [t.cpu().numpy() for t in G.fv_assemble(n, dim, kap, AG.face_velocities(n, dim, vel))]
    assert np.array_equal(got[0], rp) and np.array_equal(got[1], ci)
    assert np.array_equal(got[2].view(np.uint64), va.view(np.uint64))


@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 7, 8, 15, 16, 17, 33])
@pytest.mark.parametrize("n,dim", [(1, 2), (17, 2), (7, 3)])
def test_kappa_gradient_by_right_hand_sides(n, dim, nrhs):
    rng = np.random.default_rng(nrhs)
    N = n ** dim
    kap = 10.0 ** rng.uniform(-2, 2, N)
    lam, x = rng.uniform(-1, 1, (N, nrhs)), rng.uniform(-1, 1, (N, nrhs))
    h2 = np.longdouble(1.0) / n / n
    k, l, v = (a.astype(np.longdouble) for a in (kap, lam, x))
    ref, mag = np.zeros(N, np.longdouble), np.zeros(N, np.longdouble)
    c = np.arange(N)
    for d in range(dim):
        i = (c // n ** d) % n
        for step, inside in ((-(n ** d), i > 0), (n ** d, i < n - 1)):
            a, m = c[inside], c[inside] + step
            dT = 2 * k[m] ** 2 / ((k[a] + k[m]) ** 2 * h2)
            ref[a] += dT * ((l[a] - l[m]) * (v[a] - v[m])).sum(1)
            mag[a] += dT * (np.abs(l[a] - l[m]) * np.abs(v[a] - v[m])).sum(1)
            if d == 1:
                a = c[~inside]
                ref[a] += 2 / h2 * (l[a] * v[a]).sum(1)
                mag[a] += 2 / h2 * np.abs(l[a] * v[a]).sum(1)
    got = G.fv_kappa_grad(n, dim, kap, lam, x).cpu().numpy()
    assert np.all(np.abs(got + ref.astype(np.float64)) <= 64 * EPS * mag.astype(np.float64))


@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 7, 8, 15, 16, 17, 33])
def test_pattern_gradient_by_right_hand_sides(nrhs):
    p = W.scaled("rgg", 301, seed=1)
    rng = np.random.default_rng(nrhs)
    lam, x = rng.uniform(-1, 1, (301, nrhs)), rng.uniform(-1, 1, (301, nrhs))
    rows = np.repeat(np.arange(301), np.diff(p.rowptr))
    terms = lam.astype(np.longdouble)[rows] * x.astype(np.longdouble)[p.col]
    got = G.pattern_grad(p.rowptr, p.col, lam, x).cpu().numpy()
    assert np.all(np.abs(got + terms.sum(1).astype(np.float64)) <= 64 * EPS * np.abs(terms).sum(1).astype(np.float64))
