"""Accuracy of the tree solves where triangular factors have large inverses:
matrices far from diagonal dominance, whose factors without pivoting grow.  A
merged subtree would be solved through one dense inverse, which is then less
accurate than a substitution by its growth; such factors keep the blocks of the
dissection.  Errors against extended precision, relative to those of the level
sweeps, which substitute row by row: their geometric mean over a few matrices
stays near one (merged inverses: 20 to 216)."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_1105_3468_amd import Solver  # noqa: E402

LD = np.longdouble


def _matrix(n, seed, dominance):
    rng = np.random.default_rng(seed)
    p = W.scaled("rgg", n, seed=seed)
    a = sp.csr_matrix((p.val, p.col, p.rowptr))
    a = a - sp.diags(a.diagonal())
    a.data = rng.uniform(-1, 1, a.nnz) * 10.0 ** rng.uniform(-2, 2, a.nnz)
    rows = np.asarray(abs(a).sum(1)).ravel()
    a = (a + sp.diags(dominance * rows * rng.choice([-1, 1], n))).tocsr()
    a.sort_indices()
    return a


def _substitute(t, b, lower, unit):
    t = sp.csr_matrix(t)
    t.sort_indices()
    x = b.astype(LD).copy()
    n = len(b)
    for i in range(n) if lower else range(n - 1, -1, -1):
        q = slice(t.indptr[i], t.indptr[i + 1])
        j, v = t.indices[q], t.data[q].astype(LD)
        off = j < i if lower else j > i
        s = x[i] - (v[off] * x[j[off]]).sum()
        x[i] = s if unit else s / v[j == i][0]
    return x


def _product(m, x):
    m = sp.csr_matrix(m)
    y = np.zeros(m.shape[0], LD)
    np.add.at(y, np.repeat(np.arange(m.shape[0]), np.diff(m.indptr)), m.data.astype(LD) * x[m.indices])
    return y


def _apply(O, A, z, adjoint):
    n, nc = O.n, O.nc
    F = sp.csr_matrix((O.ilu0(), A.indices, A.indptr), shape=(n, n))
    (lr, lc, lv), (ur, uc, uv) = O.ilut()
    L0, U0 = sp.tril(F, -1) + sp.identity(n), sp.triu(F)
    L, U = sp.csr_matrix((lv, lc, lr), shape=(nc, nc)) + sp.identity(nc), sp.csr_matrix((uv, uc, ur), shape=(nc, nc))
    agg = np.asarray(O.aggregates())
    P = sp.csr_matrix((np.ones(n), (np.arange(n), agg)), shape=(n, nc))
    z = z.astype(LD)
    if not adjoint:
        t = _substitute(U0, _substitute(L0, z, True, True), False, False)
        rc = _product(P.T, z - _product(A, t))
        return t + _substitute(U, _substitute(L, rc, True, True), False, False)[agg]
    ec = _substitute(L.T, _substitute(U.T, _product(P.T, z), True, False), False, True)[agg]
    return _substitute(L0.T, _substitute(U0.T, z - _product(A.T, ec), True, False), False, True) + ec


@pytest.mark.parametrize("dominance", [0.45, 0.3])
def test_growing_factors_are_solved_in_small_blocks(dominance):
    logs = {False: [], True: []}
    for seed in range(2, 10):
        A = _matrix(1000, seed, dominance)
        opts = dict(cf=1.0, ilut_tau=0.0)
        csr = (A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
        O = oracle.Oracle(*csr, **opts)
        z = np.random.default_rng(3).uniform(-1, 1, A.shape[0])
        solvers = [Solver(*csr, **opts), Solver(*csr, sweep_kernel=1, **opts)]
        for adjoint in (False, True):
            ref = _apply(O, A, z, adjoint)
            e = [float(np.sqrt(((s.apply(z, adjoint=adjoint).cpu().numpy().astype(LD) - ref) ** 2).sum())) for s in solvers]
            logs[adjoint].append(np.log(e[0] / e[1]))
        for s in solvers:
            s.close()
    for adjoint, r in logs.items():
        assert np.exp(np.mean(r)) <= 12.0, (adjoint, np.exp(r))
