"""The single right-hand-side hop above the small-lattice limit, in each of
its boundary-phase builds (only t, any real, any complex): both daggers, every
format, with and without clover blocks, against the oracle.  The FP16 formats
go through the projection from packed words, the 12-real ones through the
fused third row.

Bars per format as in the other operator tests: 1e-12 / 1e-6 / 2e-3 / 1e-2 in
the norm."""
import numpy as np
import pytest

from oracle import clover as CL
from oracle import wilson as W
from oracle.lattice import full_to_half
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from tests._helpers import AP, ROUND, cached_gauge, link_as_stored, rel_err

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-6, "f16": 2e-3, "bf16": 1e-2}
FORMATS = [("f64", "f64", 18), ("f64", "f64", 12), ("f32", "f32", 18), ("f32", "f32", 12), ("f16", "f16", 18),
           ("f16", "f16", 12), ("bf16", "f16", 18), ("bf16", "f16", 12)]
PHASES = {"t": AP, "open-t": (1, 1, 1, 0), "real": (1, -1, 1, 0.5),
          "complex": tuple(np.exp(1j * np.array([0.4, -1.1, 2.0, 2.9])))}


@pytest.mark.parametrize("fmt_t", FORMATS, ids=lambda f: f"{f[0]}-{f[1]}-{f[2]}")
@pytest.mark.parametrize("bc", PHASES.values(), ids=PHASES.keys())
def test_hop_in_each_phase_build(bc, fmt_t):
    dims = (18, 16, 16, 16)                 # 36864 half sites
    sp, lp, reals = fmt_t
    print(f"hop phases {bc} {fmt_t}", flush=True)
    fmt, lat, ph = Format(*fmt_t), Lattice(dims, 0.124, bc), np.array(bc, dtype=np.complex128)
    u, psi, y = cached_gauge(dims, 0.5, 1800), inputs.gen_spinor_half(dims, 1801), inputs.gen_spinor_half(dims, 1802)
    blocks = inputs.gen_site_blocks(dims, 0.2, 1803)
    ai = full_to_half(np.linalg.inv(CL.blocks_to_dirac(blocks)), 1)
    u_d, x_d, y_d = lat.pack_gauge(to_device(u), fmt), *(lat.pack_spinor(to_device(q), fmt) for q in (psi, y))
    clv = lat.pack_clover(to_device(blocks), fmt)
    u_o, x_o, y_o = link_as_stored(u, lp, reals), ROUND[sp](psi), ROUND[sp](y)
    for dag in (False, True):
        h = W.hop_eo(u_o, x_o, 0, ph, dagger=dag)
        got = lat.unpack_spinor(lat.hop(u_d, x_d, fmt, 1, dagger=dag), fmt).cpu().numpy()
        assert rel_err(got, h) <= TOL[sp], dag
        got = lat.unpack_spinor(lat.hop_axpy(u_d, x_d, y_d, fmt, 1, -0.3, dagger=dag), fmt).cpu().numpy()
        assert rel_err(got, y_o - 0.3 * h) <= TOL[sp], dag
        got = lat.unpack_spinor(lat.clover_hop(u_d, clv, x_d, fmt, 1, dagger=dag), fmt).cpu().numpy()
        assert rel_err(got, CL.apply_sites(ai, h)) <= TOL[sp], (dag, "clover")
