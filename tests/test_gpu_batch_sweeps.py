"""Level sweeps over a batch of right-hand sides: the device-wide, the
one-workgroup and the mixed forms give bitwise equal solutions for every
column (they add the same terms in the same order), and every column equals
what it gives when it is the batch's only distinct one."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import Solver  # noqa: E402


@pytest.mark.parametrize("n,nrhs,fp32,order", [(5, 2, 0, 0), (301, 3, 0, 0), (301, 16, 1, 0), (3001, 2, 0, 0),
                                               (3001, 16, 0, 0), (3001, 5, 1, 2), (3001, 16, 0, 2)])
def test_batched_level_sweeps_agree(n, nrhs, fp32, order):
    p = W.scaled("rgg", n, seed=2) if n > 14 else W.scaled("fv2d", n, seed=2)
    b = np.random.default_rng(n).uniform(-1, 1, (p.n_rows, nrhs))
    b[:, -1] = b[:, 0]
    got = []
    for kern in (1, 2, 3):
        s = Solver(p.rowptr, p.col, p.val, sweep_kernel=kern, fine_order=order)
        x, r = s.solve(b, tol=1e-10, precond_fp32=fp32)
        assert r.info["converged"] == nrhs
        got.append([x.cpu().numpy()])
        if not fp32:
            got[-1].append(s.solve_adjoint(b, tol=1e-10)[0].cpu().numpy())
        s.close()
    for other in got[1:]:
        for u, v in zip(got[0], other):
            assert np.array_equal(u.view(np.uint64), v.view(np.uint64))
    for u in got[0]:
        assert np.array_equal(u[:, 0].view(np.uint64), u[:, -1].view(np.uint64))
