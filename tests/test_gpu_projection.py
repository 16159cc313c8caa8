"""The two-read projection of bases of at most 32 vectors at row counts around
its two rows a lane and 512 rows a workgroup, across the change to the
many-vector kernels at 33 vectors, and for batches: iterates after a fixed
number of steps against the oracle's modified Gram-Schmidt, within the 1e-10
of ||A dx|| / ||b|| that the parity tests use."""
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


def _chain(n):
    """A symmetric positive definite arrow on a path (one 2D-like problem for
    any row count) with strongly varying coefficients."""
    rng = np.random.default_rng(n)
    k = 10.0 ** rng.uniform(-2, 2, n)
    a = sp.diags([-k[1:], -k[1:]], [-1, 1], shape=(n, n), format="lil")
    step = max(2, int(np.sqrt(n)))
    for i in range(0, n - step):
        a[i, i + step] = a[i + step, i] = -k[i]
    a = a.tocsr()
    a = a + sp.diags(-np.asarray(a.sum(1)).ravel() + 1e-3 * k.max())
    a.sort_indices()
    return a.tocsr()


@pytest.mark.parametrize("n,steps", [(3, 3), (4, 3), (63, 12), (511, 31), (512, 32), (513, 33), (1025, 36), (1535, 40)])
def test_iterates_at_row_and_vector_edges(n, steps):
    A = _chain(n)
    rp, ci, v = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    b = np.random.default_rng(1).uniform(-1, 1, n)
    opts = dict(ilut_tau=1e-1)
    x, _ = Solver(rp, ci, v, **opts).solve(b, tol=1e-30, restart=steps, maxit=steps)
    xo, _ = oracle.Oracle(rp, ci, v, **opts).solve(b, tol=1e-30, restart=steps, maxit=steps)
    assert np.linalg.norm(A @ (x.cpu().numpy() - xo)) <= 1e-10 * np.linalg.norm(b)


@pytest.mark.parametrize("nrhs,restart", [(2, 7), (3, 30), (16, 32)])
def test_batched_iterates_match_the_oracle(nrhs, restart):
    p = W.scaled("fv2d", 23, seed=3)
    A = sp.csr_matrix((p.val, p.col, p.rowptr))
    B = np.random.default_rng(2).uniform(-1, 1, (p.n_rows, nrhs))
    X, _ = Solver(p.rowptr, p.col, p.val).solve(B, tol=1e-30, restart=restart, maxit=restart + 2)
    O = oracle.Oracle(p.rowptr, p.col, p.val)
    for c in range(nrhs):
        xo, _ = O.solve(B[:, c], tol=1e-30, restart=restart, maxit=restart + 2)
        d = A @ (X[:, c].cpu().numpy() - xo)
        assert np.linalg.norm(d) <= 1e-10 * np.linalg.norm(B[:, c])


# 32 workgroups a column, whose sums the next kernel adds, and 33, whose last
# workgroup adds them
@pytest.mark.parametrize("n", [16384, 16385])
def test_iterates_where_the_reduction_changes(n):
    A = _chain(n)
    rp, ci, v = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    B = np.random.default_rng(4).uniform(-1, 1, (n, 2))
    opts = dict(ilut_tau=1e-1)
    S, O = Solver(rp, ci, v, **opts), oracle.Oracle(rp, ci, v, **opts)
    X = S.solve(B, tol=1e-30, restart=5, maxit=7)[0].cpu().numpy()
    for c in range(2):
        x1 = S.solve(B[:, c].copy(), tol=1e-30, restart=5, maxit=7)[0].cpu().numpy()
        xo, _ = O.solve(B[:, c], tol=1e-30, restart=5, maxit=7)
        for x in (X[:, c], x1):
            assert np.linalg.norm(A @ (x - xo)) <= 1e-10 * np.linalg.norm(B[:, c])
