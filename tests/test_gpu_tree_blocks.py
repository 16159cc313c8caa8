"""Tree solves whose nodes have row counts around the 64-row blocks and
16-column slices of the blocks' inversion: 3D grids without aggregation (the
separators are grid planes, n^2 rows) and exact factors, forward and adjoint,
against the oracle entry by entry within 1e-13 of the magnitudes that flow
into each entry."""
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
from tests import _errbound as EB  # noqa: E402


@pytest.mark.parametrize("n,nrhs", [(4, 1), (7, 1), (8, 2), (9, 1), (11, 4), (12, 5), (16, 16), (18, 3)])
def test_tree_solves_at_block_edges(n, nrhs):
    p = W.scaled("fv3d", n, seed=n)
    A = sp.csr_matrix((p.val, p.col, p.rowptr))
    opts = dict(cf=1.0, ilut_tau=0.0)
    O, S = oracle.Oracle(p.rowptr, p.col, p.val, **opts), Solver(p.rowptr, p.col, p.val, **opts)
    z = p.b[:, 0]
    for adjoint in (False, True):
        ref = O.apply_adjoint(z) if adjoint else O.apply(z)
        EB.check_elementwise(S.apply(z, adjoint=adjoint).cpu().numpy(), ref, EB.apply_scale(O, A, z, adjoint=adjoint),
                             1e-13, f"n={n} adjoint={adjoint}")
    # every column of a batch like a solve of its own
    B = np.random.default_rng(n).uniform(-1, 1, (p.n_rows, nrhs))
    for solve in (S.solve, S.solve_adjoint):
        X = solve(B, tol=1e-30, restart=2, maxit=2)[0].cpu().numpy()
        for c in range(nrhs):
            x = solve(B[:, c], tol=1e-30, restart=2, maxit=2)[0].cpu().numpy()
            assert np.linalg.norm(A @ (X[:, c] - x)) <= 1e-10 * np.linalg.norm(B[:, c])
