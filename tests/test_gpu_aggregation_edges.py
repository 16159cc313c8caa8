"""Galerkin products whose aggregates' entry lists lie around the 256 pairs
that a wave sorts in LDS, and aggregates with more members than a wave has
lanes; ILU(0) of rows around the 16 lanes and 64 entries that a group of lanes
holds: aggregates, A_c and ILU(0) bit-exact against the oracle."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_1105_3468_amd import Solver  # noqa: E402


def _matrix(n, row, seed):
    """n rows of about `row` random entries (all n columns if row >= n),
    nonsymmetric, diagonally dominant."""
    rng = np.random.default_rng(seed)
    dense = row >= n
    mask = np.ones((n, n), bool) if dense else rng.random((n, n)) < row / n
    a = np.where(mask, -rng.uniform(0.1, 1.0, (n, n)), 0.0)
    np.fill_diagonal(a, 0.0)
    np.fill_diagonal(a, 1.05 * np.abs(a).sum(1) + 0.1)
    return sp.csr_matrix(a)


@pytest.mark.parametrize("n,row,cf", [(2, 2, 2.0), (40, 40, 4.0), (15, 15, 2.0), (16, 16, 2.0), (17, 17, 2.0), (63, 63, 4.0), (64, 64, 4.0), (65, 65, 4.0),
                                      (128, 128, 2.0), (129, 129, 2.0), (300, 300, 4.0), (500, 12, 100.0),
                                      (700, 3, 200.0), (1000, 6, 4.0)])
def test_lists_around_the_wave_sort(n, row, cf):
    A = _matrix(n, row, n)
    rp, ci, v = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data
    O = oracle.Oracle(rp, ci, v, cf=cf)
    S = Solver(rp, ci, v, cf=cf)
    assert np.array_equal(S.aggregates().cpu().numpy(), O.aggregates())
    for got, ref in zip(S.coarse(), O.coarse()):
        got = got.cpu().numpy()
        assert np.array_equal(got.view(np.uint64) if got.dtype == np.float64 else got,
                              ref.view(np.uint64) if ref.dtype == np.float64 else ref)
    ilu = O.ilu0()
    ref = ilu[-1] if isinstance(ilu, tuple) else ilu
    assert np.array_equal(S.ilu0().cpu().numpy().view(np.uint64), ref.view(np.uint64))
    S.close()
