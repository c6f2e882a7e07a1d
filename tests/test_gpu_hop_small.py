"""The hop kernel for lattices that leave the chip idle (8 wavefronts per 64
sites): fewer sites than lanes, ragged and whole workgroups, the last lattice
it takes and the first it does not, every format, phases, dagger, the axpy in
and out of place, norm partials and the fused dot (through solves), clover
blocks; against the oracle.

Bars per format as in the other operator tests: 1e-12 / 1e-6 / 2e-3 / 1e-2 in
the norm (its arithmetic is the single-rhs kernel's, term by term)."""
import numpy as np
import pytest

from oracle import clover as CL
from oracle import wilson as W
from oracle.lattice import full_to_half
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd import wilson_eo as WE
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from paper_2303_08609_amd.solve import cg
from tests._helpers import AP, ROUND, cached_gauge, link_as_stored, rel_err

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-6, "f16": 2e-3, "bf16": 1e-2}
FORMATS = [("f64", "f64", 18), ("f64", "f64", 12), ("f32", "f32", 18), ("f32", "f32", 12), ("f16", "f16", 18),
           ("f16", "f16", 12), ("bf16", "f16", 18), ("bf16", "f16", 12)]
CPX = tuple(np.exp(1j * np.array([0.4, -1.1, 2.0, 2.9])))
KAPPA = 0.124


@pytest.mark.parametrize("fmt_t", FORMATS, ids=lambda f: f"{f[0]}-{f[1]}-{f[2]}")
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 2, 10), (8, 4, 4, 4)], ids=lambda d: "x".join(map(str, d)))
def test_hop_and_clover(fmt_t, dims):
    sp, lp, reals = fmt_t
    print(f"small hop dims={dims} fmt={fmt_t}", flush=True)
    fmt = Format(*fmt_t)
    u = inputs.gen_gauge(dims, 0.5, 1700)
    blocks = inputs.gen_site_blocks(dims, 0.2, 1701)
    ainv = np.linalg.inv(CL.blocks_to_dirac(blocks))
    ai = [full_to_half(ainv, p) for p in (0, 1)]
    psi, y = (inputs.gen_spinor_half(dims, 1702 + q) for q in (0, 1))
    u_o, x_o, y_o = link_as_stored(u, lp, reals), ROUND[sp](psi), ROUND[sp](y)
    for bc in (AP, CPX, (1, 0, 1, -1)):
        lat, ph = Lattice(dims, KAPPA, bc), np.array(bc, dtype=np.complex128)
        u_d, x_d = lat.pack_gauge(to_device(u), fmt), lat.pack_spinor(to_device(psi), fmt)
        clv = lat.pack_clover(to_device(blocks), fmt)
        for par in (0, 1):
            for dag in (False, True):
                h = W.hop_eo(u_o, x_o, 1 - par, ph, dagger=dag)
                got = lat.unpack_spinor(lat.hop(u_d, x_d, fmt, par, dagger=dag), fmt).cpu().numpy()
                assert rel_err(got, h) <= TOL[sp], (bc, par, dag)
                y_d = lat.pack_spinor(to_device(y), fmt)
                lat.hop_axpy(u_d, x_d, y_d, fmt, par, -0.3, dagger=dag, out=y_d)
                assert rel_err(lat.unpack_spinor(y_d, fmt).cpu().numpy(), y_o - 0.3 * h) <= TOL[sp], (bc, par, dag)
                got = lat.unpack_spinor(lat.clover_hop(u_d, clv, x_d, fmt, par, dagger=dag), fmt).cpu().numpy()
                assert rel_err(got, CL.apply_sites(ai[par], h)) <= TOL[sp], (bc, par, dag, "clover")


@pytest.mark.parametrize("dims", [(16, 16, 16, 16), (16, 16, 16, 18)], ids=["last", "first-not"])
@pytest.mark.parametrize("fmt_t", [FORMATS[0], FORMATS[5]], ids=["f64-18", "f16-12"])
def test_both_sides_of_the_limit(fmt_t, dims):
    sp, lp, reals = fmt_t
    print(f"small hop limit dims={dims} fmt={fmt_t}", flush=True)
    fmt, lat = Format(*fmt_t), Lattice(dims, KAPPA, AP)
    u, psi = cached_gauge(dims, 0.5, 1710), inputs.gen_spinor_half(dims, 1711)
    got = lat.unpack_spinor(lat.apply(lat.pack_gauge(to_device(u), fmt), lat.pack_spinor(to_device(psi), fmt), fmt),
                            fmt).cpu().numpy()
    want = W.apply_m(link_as_stored(u, lp, reals), ROUND[sp](psi), KAPPA, np.array(AP, complex))
    assert rel_err(got, want) <= TOL[sp]


@pytest.mark.parametrize("method", ["cg", "bicgstab"])
@pytest.mark.parametrize("clover", [False, True], ids=["wilson", "clover"])
def test_partials_and_dots_through_solves(method, clover):
    """FP64 solves on 240 half sites: CGLS takes the norm partials, BiCGStab
    the fused dots (Wilson); the oracle's residual meets the tolerance."""
    dims, fmt = (6, 4, 2, 10), Format("f64", "f64", 18)
    print(f"small hop solve {method} clover={clover}", flush=True)
    lat = Lattice(dims, KAPPA, AP)
    u, b = inputs.gen_gauge(dims, 0.5, 1720), inputs.gen_spinor_half(dims, 1721)
    blocks = inputs.gen_site_blocks(dims, 0.2, 1722)
    x, info = cg(lat, fmt, lat.pack_gauge(to_device(u), fmt), lat.pack_spinor(to_device(b), fmt), tol=1e-11,
                 maxiter=2000, method=method, clover=lat.pack_clover(to_device(blocks), fmt) if clover else None)
    assert info["status"] == WE.WEO_OK, info
    x, ph = lat.unpack_spinor(x, fmt).cpu().numpy(), np.array(AP, complex)
    if clover:
        ainv = np.linalg.inv(CL.blocks_to_dirac(blocks))
        mx = CL.apply_m_clover(u, x, KAPPA, ph, full_to_half(ainv, 0), full_to_half(ainv, 1))
    else:
        mx = W.apply_m(u, x, KAPPA, ph)
    assert np.linalg.norm(b - mx) <= 3e-11 * np.linalg.norm(b)
