"""Products with A^T where a 256-row tile of A^T holds more entries than any tile
of A: they are staged in LDS by A^T's own tiles.  Staged products are rounded
before they are added, in column order, so the result is known bit for bit (a
lane that walks its row instead fuses the two)."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import Solver  # noqa: E402


def _matrix(n, heavy, per):
    """Tridiagonal, and `per` further rows that refer to each of the first
    `heavy` columns."""
    rng = np.random.default_rng(n)
    a = sp.diags([rng.uniform(-1, -0.5, n - 1), np.full(n, 4.0), rng.uniform(-1, -0.5, n - 1)], [-1, 0, 1]).tolil()
    for j in range(heavy):
        for i in rng.choice(np.arange(300, n), per, replace=False):
            a[i, j] = rng.uniform(-0.05, 0.05)
    a = a.tocsr()
    a.sort_indices()
    return a


def _rows_added_in_order(m, x):
    p = m.data * x[m.indices]
    y = np.zeros(m.shape[0])
    for i in range(m.shape[0]):
        for q in range(m.indptr[i], m.indptr[i + 1]):
            y[i] = y[i] + p[q]
    return y


# entries of A^T's first tile: below 2048, between the two capacities, beyond
@pytest.mark.parametrize("per", [5, 40, 120])
def test_transposed_product_by_its_own_tiles(per):
    n = 4000
    A = _matrix(n, 40, per)
    AT = A.T.tocsr()
    AT.sort_indices()

    def most(m):
        return max(m.indptr[min(n, r + 256)] - m.indptr[r] for r in range(0, n, 256))

    assert most(A) <= 2048
    x = np.random.default_rng(1).uniform(-1, 1, n)
    s = Solver(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    xd = torch.as_tensor(x, device="cuda")
    for m, transposed in ((A, False), (AT, True)):
        y = s.spmv(xd, transposed=transposed).cpu().numpy()
        ref = _rows_added_in_order(m, x)
        if most(m) <= 4096:
            assert np.array_equal(y.view(np.uint64), ref.view(np.uint64)), (transposed, most(m))
        assert np.all(np.abs(y - ref) <= 256 * 2.0 ** -53 * (abs(m) @ np.abs(x)))
    s.close()
