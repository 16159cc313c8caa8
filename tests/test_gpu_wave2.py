"""Wavefront sweeps of fine factors with 2D-grid structure at the edges of
their layout: bands of 64 grid rows, chunks of 8 steps, and the result's turn
back to cell order in tiles of 16 steps.  The sweeps perform the operations of
the level sweeps (sweep_kernel 1) in the same order, so applications agree
bitwise, singly and as columns of a batch, whose right-hand sides are read in
cell order, and repeated ones, between which what the sweeps poll is reset."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import Solver  # noqa: E402


def _grid5(nx, ny, seed):
    rng = np.random.default_rng(seed)
    n = nx * ny
    k = np.arange(n).reshape(ny, nx)
    i = np.concatenate([k[:, :-1].ravel(), k[:-1].ravel()])
    j = np.concatenate([k[:, 1:].ravel(), k[1:].ravel()])
    a = sp.coo_matrix((-rng.uniform(0.1, 1, 2 * len(i)), (np.r_[i, j], np.r_[j, i])), (n, n)).tocsr()
    a = (a + sp.diags(-np.asarray(a.sum(1)).ravel() + 0.1)).tocsr()
    a.sort_indices()
    return a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data


@pytest.mark.parametrize("nx,ny", [(3, 200), (17, 63), (16, 64), (33, 65), (65, 128), (300, 130), (1, 70), (128, 129), (200, 3)])
def test_wave2_bitwise_equal_to_level_sweeps(nx, ny):
    A = _grid5(nx, ny, nx)
    n = nx * ny
    S3, S1 = Solver(*A, sweep_kernel=3), Solver(*A, sweep_kernel=1)
    rng = np.random.default_rng(5)
    for prec, adj in ((0, False), (1, False), (0, True)):
        for _ in range(2):
            z = torch.as_tensor(rng.uniform(-1, 1, n), device="cuda")
            assert torch.equal(S3.apply(z, precision=prec, adjoint=adj), S1.apply(z, precision=prec, adjoint=adj))
    B = rng.uniform(-1, 1, (n, 3))
    for prec in (0, 1):
        X3, X1 = (S.solve(B, tol=1e-30, maxit=3, precond_fp32=bool(prec))[0] for S in (S3, S1))
        assert torch.equal(X3, X1)
