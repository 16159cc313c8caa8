"""Several right-hand sides where their kernels can go wrong: systems of one to
nine rows and batches that end with a single column; tree solves of several
columns in FP32, and of the transpose, at the edges of the inverses' blocks; and
a matrix whose one wide row or column sends its setup down the general paths."""
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


def _csr(A):
    A = sp.csr_matrix(A)
    A.sort_indices()
    return A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data


@pytest.mark.parametrize("nrhs", [2, 5, 17])
@pytest.mark.parametrize("n", [1, 2, 3, 9])
def test_a_handful_of_rows(n, nrhs):
    rng = np.random.default_rng(n)
    a = -rng.uniform(0.1, 1.0, (n, n))
    np.fill_diagonal(a, 0.0)
    np.fill_diagonal(a, 1.1 * np.abs(a).sum(1) + 0.1)
    B = rng.uniform(-1, 1, (n, nrhs))
    B[:, -1] = B[:, 0]
    S = Solver(*_csr(a), cf=1.0 if n < 3 else 2.0)
    for m, run in ((a, lambda: S.solve(B, tol=1e-10)), (a.T, lambda: S.solve_adjoint(B, tol=1e-10)),
                   (a, lambda: S.solve(B, tol=1e-10, precond_fp32=1))):
        X, r = run()
        X = X.cpu().numpy()
        assert r.info["converged"] == nrhs
        assert np.all(np.linalg.norm(m @ X - B, axis=0) <= 1e-10 * np.linalg.norm(B, axis=0))
        if nrhs <= 16:  # columns of one batch
            assert np.array_equal(X[:, -1].view(np.uint64), X[:, 0].view(np.uint64))


# separators of n^2 rows around the 16-row slices and the 64-row blocks
@pytest.mark.parametrize("n,nrhs", [(4, 3), (5, 16), (8, 2), (9, 5), (11, 16), (16, 4), (17, 8)])
def test_columns_at_block_edges(n, nrhs):
    p = W.scaled("fv3d", n, seed=n)
    A = sp.csr_matrix((p.val, p.col, p.rowptr))
    S = Solver(p.rowptr, p.col, p.val, cf=1.0, ilut_tau=0.0)
    B = np.random.default_rng(n).uniform(-1, 1, (p.n_rows, nrhs))
    # FP32 cycles round at 6e-8 in every term of sums of up to a few hundred
    for M, solve, tol in ((A.T.tocsr(), S.solve_adjoint, 1e-10),
                          (A, lambda b, **kw: S.solve(b, precond_fp32=1, **kw), 1e-4)):
        X = solve(B, tol=1e-30, restart=2, maxit=2)[0].cpu().numpy()
        for c in range(nrhs):
            x = solve(B[:, c].copy(), tol=1e-30, restart=2, maxit=2)[0].cpu().numpy()
            assert np.linalg.norm(M @ (X[:, c] - x)) <= tol * np.linalg.norm(B[:, c])


@pytest.mark.parametrize("wide", ["row", "column", "both"])
def test_one_wide_row(wide):
    """300 entries in one row (column) of a matrix of 5 to 9 a row: aggregates,
    A_c and ILU(0) by a thread per list and row, bit for bit."""
    n = 2000
    p = W.scaled("rgg", n, seed=6)
    A = sp.csr_matrix((p.val, p.col, p.rowptr)).tolil()
    rng = np.random.default_rng(7)
    at = rng.choice(np.setdiff1d(np.arange(n), [1000]), 300, replace=False)
    for j in at:
        if wide in ("row", "both"):
            A[1000, j] = -rng.uniform(0.01, 0.02)
        if wide in ("column", "both"):
            A[j, 1000] = -rng.uniform(0.01, 0.02)
    A = A.tocsr()
    A = A + sp.diags(np.asarray(abs(A).sum(1)).ravel() - A.diagonal())
    csr = _csr(A)
    O, S = oracle.Oracle(*csr), Solver(*csr)
    assert np.array_equal(S.aggregates().cpu().numpy(), O.aggregates())
    for got, ref in zip(S.coarse(), O.coarse()):
        got = got.cpu().numpy()
        assert got.tobytes() == np.ascontiguousarray(ref, dtype=got.dtype).tobytes()
    assert S.ilu0().cpu().numpy().tobytes() == O.ilu0().tobytes()
    b = rng.uniform(-1, 1, n)
    x, r = S.solve(b, tol=1e-10)
    assert r.info["converged"] == 1 and np.linalg.norm(A @ x.cpu().numpy() - b) <= 1e-10 * np.linalg.norm(b)
