"""The solve's status block (masks, flags, norms read in one copy): one and
the largest number of right-hand sides, of which some are done from the start
(zero source; a start that meets the tolerance), for each method that keeps
masks, plain and mixed, and M^dag M (whose mixed solve keeps converged
right-hand sides in their slots).

Bar: the oracle's FP64 residual of each right-hand side within 1.05 of the
tolerance; zero sources give exactly zero."""
import numpy as np
import pytest

from oracle import wilson as W
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd import wilson_eo as WE
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from paper_2303_08609_amd.solve import cg
from tests._helpers import AP

pytestmark = pytest.mark.gpu

DIMS, KAPPA, TOL = (4, 4, 4, 6), 0.12, 1e-10
F64 = Format("f64", "f64", 18)
PH = np.array(AP, dtype=np.complex128)


def _a(u, x, op):
    y = W.apply_m(u, x, KAPPA, PH)
    return W.apply_m(u, y, KAPPA, PH, dagger=True) if op == "MdagM" else y


@pytest.mark.parametrize("nrhs", [1, 2, 16])
@pytest.mark.parametrize("inner", [None, "f32", "f16", "bf16"])
@pytest.mark.parametrize("op,method", [("M", "bicgstab"), ("M", "cg"), ("MdagM", "cg"), ("MdagM", "bicgstab")])
def test_done_and_live_together(op, method, inner, nrhs):
    print(f"status {op} {method} inner={inner} nrhs={nrhs}", flush=True)
    lat = Lattice(DIMS, KAPPA, AP)
    u = inputs.gen_gauge(DIMS, 0.3, 2000)
    u_p = lat.pack_gauge(to_device(u), F64)
    b = inputs.gen_spinor_half(DIMS, 2001, nrhs=nrhs)
    b[nrhs // 2 + 1::5] = 0.0                                   # zero sources
    pack = lambda v: lat.pack_spinor(to_device(v), F64)
    get = lambda p: lat.unpack_spinor(p, F64, nrhs=nrhs).cpu().numpy().reshape(b.shape)
    kw = dict(nrhs=nrhs, op=op, tol=TOL, maxiter=4000, method=method)
    if inner:
        fi = Format(inner, "f32" if inner == "f32" else "f16", 12)
        kw.update(inner=fi, u_inner=lat.pack_gauge(to_device(u), fi), inner_tol=1e-2)
    b_p = pack(b) if nrhs > 1 else pack(b[0])
    x_p, info = cg(lat, F64, u_p, b_p, **kw)
    assert info["status"] == WE.WEO_OK, info
    x = get(x_p)
    x0 = np.zeros_like(b)
    x0[::3] = x[::3]                                            # converged starts
    x2, info2 = cg(lat, F64, u_p, b_p, x0=pack(x0) if nrhs > 1 else pack(x0[0]), **kw)
    assert info2["status"] == WE.WEO_OK, info2
    if nrhs == 1:
        assert info2["iters"] == 0
    x2 = get(x2)
    for q in (x, x2):
        for r in range(nrhs):
            if not b[r].any():
                assert not q[r].any(), r
            else:
                assert np.linalg.norm(_a(u, q[r], op) - b[r]) <= 1.05 * TOL * np.linalg.norm(b[r]), r
