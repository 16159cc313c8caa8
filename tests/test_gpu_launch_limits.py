"""Gradients of so many rows that several lanes a row would be more threads than
a launch along x may have (2^32 - 1): fewer lanes share a row then."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import gmg as G  # noqa: E402


def _room(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip("not enough device memory")


def test_pattern_gradient_of_many_rows():
    n, nrhs = (1 << 28) + 5, 16
    _room(48)
    x = torch.empty((n, nrhs), device="cuda", dtype=torch.float64)
    x[:] = torch.arange(1, nrhs + 1, device="cuda", dtype=torch.float64)
    x[-1] = 0.5
    rp = torch.arange(n + 1, device="cuda", dtype=torch.int32)
    g = G.pattern_grad(rp, rp[:-1], x, x)
    assert float(g[-1]) == -4.0
    assert bool((g[:-1] == -float(sum(k * k for k in range(1, nrhs + 1)))).all())


def test_kappa_gradient_of_many_cells():
    n, nrhs = 646, 16
    _room(48)
    N = n ** 3
    x = torch.ones((N, nrhs), device="cuda", dtype=torch.float64)
    kap = torch.ones(N, device="cuda", dtype=torch.float64)
    g = G.fv_kappa_grad(n, 3, kap, x, x).view(n, n, n)  # z, y, x
    # equal values on both sides of every inner face: the Dirichlet faces remain
    assert bool((g[:, 1:-1] == 0).all())
    h = 1.0 / n
    face = -(2.0 / (h * h)) * nrhs
    for j in (0, n - 1):
        assert float((g[:, j] - face).abs().max()) <= 64 * 2.0 ** -52 * abs(face)
