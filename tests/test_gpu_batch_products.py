"""Sparse products of a batch at the row counts where the columns that share a
workgroup change (64 and 65, 255 and 256 workgroups of 256 rows): iterates of
every column against the single solve, whose products are another kernel,
within the 1e-10 of ||A dx|| / ||b|| that the parity tests use; a column
repeated in another group is bitwise equal."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import Solver  # noqa: E402


@pytest.mark.parametrize("n", [9, 16384, 16385, 65280, 65281])
def test_columns_match_single_solves(n):
    p = W.scaled("rgg", max(n, 15), seed=3)
    A = sp.csr_matrix((p.val, p.col, p.rowptr))
    m = A.shape[0]
    B = np.random.default_rng(n).uniform(-1, 1, (m, 5))
    B[:, 4] = B[:, 0]
    S = Solver(p.rowptr, p.col, p.val)
    for solve, M in ((S.solve, A), (S.solve_adjoint, A.T.tocsr())):
        X = solve(B, tol=1e-30, maxit=6)[0].cpu().numpy()
        assert np.array_equal(X[:, 4].view(np.uint64), X[:, 0].view(np.uint64))
        for c in range(4):
            x = solve(B[:, c].copy(), tol=1e-30, maxit=6)[0].cpu().numpy()
            assert np.linalg.norm(M @ (X[:, c] - x)) <= 1e-10 * np.linalg.norm(B[:, c])
