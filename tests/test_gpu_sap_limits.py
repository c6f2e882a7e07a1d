"""SAP block shapes next to the limit sum 1 / b_mu <= 2 over the cut directions
that separates the two sweep kernels: exactly 2 with all directions cut and
with two extents of 1, one extent of 1 on either side, against the oracle.

Bars as for the other block shapes: 1e-5 relative in the norm, 1e-4 per site
(at most 9 MR steps of some hundred FP32 operations per component)."""
import numpy as np
import pytest

from oracle import sap as OS
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from tests._helpers import ROUND, link_as_stored, rel_err, site_rel_max
from tests.test_gpu_sap import _full_field, _unpack_full

pytestmark = pytest.mark.gpu

CPX = tuple(np.exp(1j * np.array([0.4, -1.1, 2.0, 2.9])))
CASES = [
    # dims, block, link reals                         sum 1 / b
    ((4, 4, 4, 4), (2, 2, 2, 2), 18),               # 2
    ((4, 4, 2, 4), (1, 1, 2, 4), 12),               # 2; z and t spanned
    ((4, 8, 4, 8), (1, 4, 2, 4), 18),               # 2; one extent of 1
    ((4, 8, 8, 8), (1, 4, 4, 4), 12),               # 1.75
    ((4, 4, 4, 8), (1, 2, 2, 4), 18),               # 2.25: the general kernel
    ((4, 4, 4, 4), (1, 2, 2, 2), 12),               # 2.5: the general kernel
]


@pytest.mark.parametrize("dims, block, reals", CASES, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else c)
def test_sap_near_the_face_limit(dims, block, reals):
    print(f"SAP face limit dims={dims} block={block}", flush=True)
    fmt, nrhs, ncy, nmr = Format("f32", "f32", reals), 2, 3, 3
    lat = Lattice(dims, 0.124, CPX)
    u = inputs.gen_gauge(dims, 0.5, 2200 + sum(dims))
    eta = np.stack([inputs.gen_spinor_full(dims, 2201 + r) for r in range(nrhs)])
    u_d, e_d = lat.pack_gauge(to_device(u), fmt), _full_field(lat, fmt, eta, nrhs=nrhs)
    got = _unpack_full(lat, fmt, lat.sap(u_d, e_d, fmt, block, ncy, nmr, nrhs=nrhs), nrhs=nrhs)
    for r in range(nrhs):
        want = OS.sap(link_as_stored(u, "f32", reals), ROUND["f32"](eta[r]), 0.124, np.array(CPX), block, ncy, nmr)
        assert rel_err(got[r], want) <= 1e-5 and site_rel_max(got[r], want) <= 1e-4, r
