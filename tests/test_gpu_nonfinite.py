"""Infinities stay where they belong: the tree solves multiply by dense inverses
of several subtrees at once, and a zero entry of an inverse must not turn
another part's infinity into a NaN.  Systems of several parts that do not know
of each other: a part with an infinity in its right-hand side leaves the others
as they are without it."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import Solver  # noqa: E402


def _parts(name):
    def m(kind, n):
        p = W.scaled(kind, n)
        return sp.csr_matrix((p.val, p.col, p.rowptr))

    return {"grids": [m("fv2d", 12), m("fv2d", 17), m("fv3d", 6)], "graphs": [m("rgg", 300)] * 5,
            "large": [m("fv2d", 60), m("rgg", 1500)]}[name]


@pytest.mark.parametrize("cf", [4.0, 1.0])
@pytest.mark.parametrize("name", ["grids", "graphs", "large"])
def test_infinity_stays_in_its_part(name, cf):
    parts = _parts(name)
    A = sp.block_diag(parts, format="csr")
    A.sort_indices()
    ends = np.cumsum([p.shape[0] for p in parts])
    S = Solver(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, cf=cf)
    z = np.random.default_rng(1).uniform(-1, 1, A.shape[0])
    for kw, tol in ((dict(), 1e-12), (dict(adjoint=True), 1e-12), (dict(precision=1), 1e-5)):
        ref = S.apply(torch.as_tensor(z, device="cuda"), **kw).cpu().numpy()
        for k, end in enumerate(ends):
            start = end - parts[k].shape[0]
            bad = z.copy()
            bad[(start + end) // 2] = np.inf
            q = S.apply(torch.as_tensor(bad, device="cuda"), **kw).cpu().numpy()
            assert not np.isfinite(q[start:end]).all()
            others = np.r_[0:start, end:A.shape[0]]
            assert np.linalg.norm(q[others] - ref[others]) <= tol * np.linalg.norm(ref[others]), (kw, k)
            # and nothing is left behind
            again = S.apply(torch.as_tensor(z, device="cuda"), **kw).cpu().numpy()
            assert np.array_equal(again.view(np.uint64), ref.view(np.uint64))


def test_overflow_of_an_inverse_stays_in_its_part():
    """A chain whose exact factor's inverse overflows, beside a grid that is
    solved together with it."""
    n = 40
    chain = sp.diags([np.full(n - 1, 1e40), np.full(n, 1.0)], [-1, 0], format="csr")
    p = W.scaled("fv2d", 9)
    grid = sp.csr_matrix((p.val, p.col, p.rowptr))
    opts = dict(cf=1.0, ilut_tau=0.0)
    alone = Solver(grid.indptr.astype(np.int32), grid.indices.astype(np.int32), grid.data, **opts)
    z = np.random.default_rng(1).uniform(-1, 1, n + grid.shape[0])
    for parts in ([chain, grid], [grid, chain]):
        A = sp.block_diag(parts, format="csr")
        A.sort_indices()
        rows = slice(n, None) if parts[0] is chain else slice(0, grid.shape[0])
        S = Solver(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, **opts)
        for adjoint in (False, True):
            q = S.apply(torch.as_tensor(z, device="cuda"), adjoint=adjoint).cpu().numpy()[rows]
            ref = alone.apply(torch.as_tensor(z[rows], device="cuda"), adjoint=adjoint).cpu().numpy()
            assert np.linalg.norm(q - ref) <= 1e-11 * np.linalg.norm(ref)
