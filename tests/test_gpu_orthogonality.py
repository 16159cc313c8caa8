"""Orthogonality of the FGMRES basis.  The projection kernels are driven
directly, as the solver drives them, with an operator I + delta E: a step then
cancels all but delta of its vector, and one projection alone would leave
products of eps / delta in the basis.  Two projections leave the rounding of the
products themselves, n u |v| |v| at most (u = 2^-53); the column returned to the
host must rebuild the vector it came from to as much."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1105_3468_amd import gmg  # noqa: E402

P, L, I = C.c_void_p, C.c_size_t, C.c_int


class BatchCols(C.Structure):
    _fields_ = [("nb", I), ("vcol", L), ("wcol", L), ("rcol", L), ("hcol", L), ("fcol", L)]


def _kernels():
    lib = gmg.load()

    def get(name, *args):
        f = lib[name]
        f.restype, f.argtypes = None, list(args)
        return f

    return (get("_ZN3gmg8red_initERNS_7RedWorkEP12ihipStream_t", P, P),
            get("_ZN3gmg15launch_multidotEPdmiPKdS2_lRNS_7RedWorkES0_P12ihipStream_tRKNS_9BatchColsE",
                P, L, I, P, P, C.c_int64, P, P, P, P),
            get("_ZN3gmg13launch_updateEPKdmiPdS2_lRNS_7RedWorkES2_P12ihipStream_tRKNS_9BatchColsE",
                P, L, I, P, P, C.c_int64, P, P, P, P),
            get("_ZN3gmg16launch_normalizeEPKdPdliS1_S2_S2_mS1_S2_RNS_7RedWorkEP12ihipStream_tRKNS_9BatchColsE",
                P, P, C.c_int64, I, P, P, P, L, P, P, P, P, P),
            get("_ZN3gmg12launch_againEPdmiPKdlP12ihipStream_t", P, L, I, P, C.c_int64, P))


# 700 rows: sums added by the next kernel; 40001: by the last block
@pytest.mark.parametrize("n,nb", [(700, 1), (701, 3), (40001, 1), (40000, 2)])
@pytest.mark.parametrize("delta", [1.0, 1e-5, 1e-9])
def test_basis_stays_orthonormal(n, nb, delta):
    red_init, multidot, update, normalize, again = _kernels()
    steps, fcol, hcol = 32, 33, 72
    g = torch.Generator(device="cuda").manual_seed(n)

    def new(*shape):
        return torch.zeros(shape, device="cuda", dtype=torch.float64)

    ld = (n + 63) // 64 * 64
    V, w, h, dots, fix = new(steps + 1, nb, ld), new(nb, ld), new(nb, hcol), new(nb, fcol), new(nb, fcol)
    host = torch.zeros((nb, hcol), dtype=torch.float64).pin_memory()
    d = torch.rand((nb, n), generator=g, device="cuda", dtype=torch.float64) * 2 - 1
    V[0, :, :n] = torch.rand((nb, n), generator=g, device="cuda", dtype=torch.float64) - 0.5
    V[0] /= V[0].norm(dim=1, keepdim=True)
    work = C.create_string_buffer(4096)  # the reductions' scratch, kept until the process ends
    s = torch.cuda.current_stream().cuda_stream
    red_init(work, s)
    cd, cf = BatchCols(nb, ld, ld, hcol, hcol, fcol), BatchCols(nb, ld, ld, fcol, hcol, fcol)
    ws, cols = [], []
    for k in range(1, steps + 1):
        v = V[k - 1, :, :n]
        w[:, :n] = v + delta * d * v.roll(1, 1)
        ws.append(w[:, :n].clone())
        multidot(V.data_ptr(), nb * ld, k, fix.data_ptr(), w.data_ptr(), n, work, h.data_ptr(), s, C.byref(cd))
        update(V.data_ptr(), nb * ld, k, h.data_ptr(), w.data_ptr(), n, work, dots.data_ptr(), s, C.byref(cf))
        normalize(w.data_ptr(), V[k].data_ptr(), n, k, dots.data_ptr(), fix.data_ptr(), None, 0, h.data_ptr(),
                  host.data_ptr(), work, s, C.byref(cf))
        torch.cuda.synchronize()
        cols.append(torch.cat([host[:, :k] + host[:, k:2 * k], host[:, 2 * k:2 * k + 1].sqrt()], 1).cuda())
    if nb == 1:
        again(V.data_ptr(), ld, steps, fix.data_ptr(), n, s)
    torch.cuda.synchronize()
    tol = n * 2.0 ** -53
    last = steps + 1 if nb == 1 else steps  # vectors projected twice
    for c in range(nb):
        B = V[:last, c, :n]
        off = (B @ B.T - torch.eye(last, device="cuda", dtype=torch.float64)).abs().max()
        assert float(off) <= tol, float(off)
        for k in range(1, last):
            err = (ws[k - 1][c] - cols[k - 1][c] @ B[:k + 1]).norm()
            assert float(err) <= tol, (k, float(err))
