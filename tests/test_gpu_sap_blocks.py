"""Block shapes of the SAP sweep where its kernels change: 64, 128 and 256
lanes, blocks that leave lanes idle (3^4), the solution kept in block order
(sum 1 / b_mu <= 1 over the cut directions) or in lattice order (<= 2), the
general kernel (> 2), one and several cycles, spanned directions with and
without a phase, two right-hand sides; against the oracle.

Bar: relative 1e-5 norm-wise, 1e-4 per site.  Each MR step is a hop (a few
hundred FP32 operations per component, rounding 6e-8 each, adding as their
square root) and its step sizes depend on the data; at most 15 steps follow
each other here: 15 * 20 * 6e-8 = 2e-5 at the worst site, ten times below the
per-site bar, and a tenth of that in the norm.
"""
import numpy as np
import pytest
import torch

from oracle import sap as OS
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from tests._helpers import ROUND, link_as_stored, rel_err, site_rel_max
from tests.test_gpu_sap import _full_field, _unpack_full

pytestmark = pytest.mark.gpu

CPX = tuple(np.exp(1j * np.array([0.4, -1.1, 2.0, 2.9])))
AP = (1, 1, 1, -1)
CASES = [
    # dims, block, ncy, nmr, link reals, phases
    ((6, 6, 6, 6), (3, 3, 3, 3), 2, 3, 18, CPX),      # 81 of 128 lanes; lattice order
    ((8, 6, 6, 4), (4, 3, 3, 4), 3, 3, 12, CPX),      # 144 of 256 lanes; t spanned with a phase; block order
    ((8, 8, 4, 4), (4, 4, 4, 4), 1, 4, 18, AP),       # one cycle; z spanned without, t with a phase
    ((8, 8, 8, 4), (4, 4, 4, 4), 3, 2, 12, (1, 1, 1, 1)),
    ((16, 8, 4, 4), (8, 4, 2, 4), 2, 3, 18, AP),      # 256 lanes, sum 1 / b = 0.875
    ((8, 4, 4, 4), (2, 4, 2, 2), 2, 3, 12, CPX),      # 32 of 64 lanes, sum 1 / b = 1.5
    ((4, 4, 4, 4), (1, 1, 2, 4), 2, 3, 18, CPX),      # sum 1 / b = 2.5: the general kernel
    ((4, 4, 4, 4), (1, 1, 1, 1), 3, 1, 12, AP),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{'x'.join(map(str, c[0]))}-b{''.join(map(str, c[1]))}")
def test_sap_block_shapes(case):
    dims, block, ncy, nmr, reals, ph = case
    print(f"SAP blocks dims={dims} block={block}", flush=True)
    fmt, nrhs = Format("f32", "f32", reals), 2
    lat = Lattice(dims, 0.124, ph)
    u = inputs.gen_gauge(dims, 0.5, 1400 + sum(dims))
    eta = np.stack([inputs.gen_spinor_full(dims, 1401 + r) for r in range(nrhs)])
    u_d, e_d = lat.pack_gauge(to_device(u), fmt), _full_field(lat, fmt, eta, nrhs=nrhs)
    psi = lat.sap(u_d, e_d, fmt, block, ncy, nmr, nrhs=nrhs)
    assert torch.equal(psi, lat.sap(u_d, e_d, fmt, block, ncy, nmr, nrhs=nrhs))
    got = _unpack_full(lat, fmt, psi, nrhs=nrhs)
    for r in range(nrhs):
        want = OS.sap(link_as_stored(u, "f32", reals), ROUND["f32"](eta[r]), 0.124, np.array(ph, complex), block,
                      ncy, nmr)
        e, m = rel_err(got[r], want), site_rel_max(got[r], want)
        print(f"  rhs {r}: norm-wise {e:.2e}, per site {m:.2e}", flush=True)
        assert e <= 1e-5 and m <= 1e-4
