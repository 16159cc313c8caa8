"""Scheduling of the device-wide level sweeps: `sweep_waves` bounds the waves
that sweep, and sweeps of two solvers that overlap on one device both finish,
with the bits of solves run alone."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import Solver  # noqa: E402


def test_few_waves_sweep_with_few_waves():
    """One workgroup takes its chunks one group after another: 2500 chunks with
    4 waves take far longer than with a thousand waves."""
    p = W.scaled("rgg", 20000, seed=4)
    z = torch.as_tensor(np.random.default_rng(1).uniform(-1, 1, p.n_rows), device="cuda")
    us = {}
    ref = None
    for w in (4, 64, 1024, 4096):
        s = Solver(p.rowptr, p.col, p.val, sweep_kernel=1, sweep_waves=w)
        s.apply(z)
        s.profile(True, classes=["sweep_fine"])
        q = s.apply(z)
        r = s.profile_read()["sweep_fine"]
        us[w] = 1e3 * r["ms"] / r["launches"]
        ref = q if ref is None else ref
        assert torch.equal(q, ref), w
        s.close()
    print(us)
    assert us[4] > 3 * us[64] and us[4] > 3 * us[1024], us


@pytest.mark.parametrize("waves", [0, 16, 8192])
def test_overlapping_sweeps(waves):
    ps = [W.scaled("rgg", 20000, seed=4), W.scaled("fv2d", 120, seed=2)]
    streams = [torch.cuda.Stream() for _ in ps]
    rng = np.random.default_rng(2)
    bs = [torch.as_tensor(rng.uniform(-1, 1, (p.n_rows, 3)), device="cuda") for p in ps]
    torch.cuda.synchronize()
    solvers = []
    for p, st in zip(ps, streams):
        with torch.cuda.stream(st):
            solvers.append(Solver(p.rowptr, p.col, p.val, sweep_kernel=1, sweep_waves=waves, stream=st))

    def solve(i):
        with torch.cuda.stream(streams[i]):
            x, r = solvers[i].solve(bs[i], tol=1e-9, restart=30, maxit=60)
            streams[i].synchronize()
            return x.clone(), r.info["iters"]

    alone = [solve(i) for i in range(2)]
    got, errs = [None, None], []

    def work(i):
        try:
            got[i] = [solve(i) for _ in range(3)]
        except Exception as e:  # reported by the test's own thread
            errs.append(e)

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not errs, errs
    for i in range(2):
        for x, it in got[i]:
            assert it == alone[i][1] and torch.equal(x, alone[i][0])
    for s in solvers:
        s.close()
