"""The single right-hand-side hop kernels above the small-lattice limit on a
lattice that fills no whole workgroups (18 x 14 x 18 x 18: 40824 half sites,
120 in the last workgroup of 256, 56 in its last wavefront): hop, axpy, clover
hop and clover apply in every format at every site, and the last norm and dot
partials through solves.

Bars per format as in the other operator tests, 1e-12 / 1e-6 / 2e-3 / 1e-2
relative in the norm, and per site 1e-11 / 1e-5 / 1e-2 / 5e-2 (a site's 12
components scatter more than the norm of the field); solves to a true residual
of 2e-8 for a tolerance of 1e-8."""
import numpy as np
import pytest

from oracle import clover as CL
from oracle import wilson as W
from oracle.lattice import full_to_half
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd import wilson_eo as WE
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from paper_2303_08609_amd.solve import cg
from tests._helpers import AP, ROUND, cached_gauge, link_as_stored, rel_err, site_rel_max

pytestmark = pytest.mark.gpu

DIMS, KAPPA, PH = (18, 14, 18, 18), 0.122, np.array(AP, dtype=np.complex128)
TOL = {"f64": 1e-12, "f32": 1e-6, "f16": 2e-3, "bf16": 1e-2}
SITE = {"f64": 1e-11, "f32": 1e-5, "f16": 1e-2, "bf16": 5e-2}
FORMATS = [("f64", "f64", 18), ("f64", "f64", 12), ("f32", "f32", 18), ("f32", "f32", 12), ("f16", "f16", 18),
           ("f16", "f16", 12), ("bf16", "f16", 18), ("bf16", "f16", 12)]


def _blocks():
    blocks = inputs.gen_site_blocks(DIMS, 0.2, 2103)
    return blocks, np.linalg.inv(CL.blocks_to_dirac(blocks))


@pytest.mark.parametrize("fmt_t", FORMATS, ids=lambda f: f"{f[0]}-{f[1]}-{f[2]}")
def test_hops_and_clover(fmt_t):
    sp, lp, reals = fmt_t
    print(f"hop remainders {fmt_t}", flush=True)
    fmt, lat = Format(*fmt_t), Lattice(DIMS, KAPPA, AP)
    u, psi, y = cached_gauge(DIMS, 0.5, 2100), *(inputs.gen_spinor_half(DIMS, 2101 + q) for q in (0, 1))
    blocks, ainv = _blocks()
    ai = [full_to_half(ainv, p) for p in (0, 1)]
    u_d, x_d, y_d = lat.pack_gauge(to_device(u), fmt), *(lat.pack_spinor(to_device(q), fmt) for q in (psi, y))
    clv = lat.pack_clover(to_device(blocks), fmt)
    u_o, x_o, y_o = link_as_stored(u, lp, reals), ROUND[sp](psi), ROUND[sp](y)

    def check(got, want, what):
        got = lat.unpack_spinor(got, fmt).cpu().numpy()
        assert rel_err(got, want) <= TOL[sp] and site_rel_max(got, want) <= SITE[sp], what

    for dag in (False, True):
        h = W.hop_eo(u_o, x_o, 0, PH, dagger=dag)
        check(lat.hop(u_d, x_d, fmt, 1, dagger=dag), h, (dag, "hop"))
        check(lat.hop_axpy(u_d, x_d, y_d, fmt, 1, -0.3, dagger=dag), y_o - 0.3 * h, (dag, "axpy"))
        check(lat.clover_hop(u_d, clv, x_d, fmt, 1, dagger=dag), CL.apply_sites(ai[1], h), (dag, "clover hop"))
        check(lat.clover_apply(u_d, clv, x_d, fmt, dagger=dag),
              CL.apply_m_clover(u_o, x_o, KAPPA, PH, ai[0], ai[1], dagger=dag), (dag, "clover apply"))


@pytest.mark.parametrize("method, clover", [("cg", False), ("bicgstab", False), ("cg", True)])
def test_norm_and_dot_partials(method, clover):
    print(f"hop remainders in a solve: {method} clover={clover}", flush=True)
    fmt, lat = Format("f64", "f64", 18), Lattice(DIMS, KAPPA, AP)
    u, b = cached_gauge(DIMS, 0.5, 2100), inputs.gen_spinor_half(DIMS, 2102)
    u_d, b_d = lat.pack_gauge(to_device(u), fmt), lat.pack_spinor(to_device(b), fmt)
    kw, op = {}, lambda x: W.apply_m(u, x, KAPPA, PH)
    if clover:
        blocks, ainv = _blocks()
        kw["clover"] = lat.pack_clover(to_device(blocks), fmt)
        ai = [full_to_half(ainv, p) for p in (0, 1)]
        op = lambda x: CL.apply_m_clover(u, x, KAPPA, PH, ai[0], ai[1])
    x_d, info = cg(lat, fmt, u_d, b_d, tol=1e-8, maxiter=1000, method=method, **kw)
    assert info["status"] == WE.WEO_OK, info
    res = b - op(lat.unpack_spinor(x_d, fmt).cpu().numpy())
    assert np.linalg.norm(res) <= 2e-8 * np.linalg.norm(b)
