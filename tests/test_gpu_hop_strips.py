"""The single right-hand-side hop walked in z strips (lattices whose t slices
outgrow an XCD's L2): both strip rules, strips that end in a partly filled
workgroup, norm partials where strips are multiples of 64 sites and where they
are not.  Every site against the multi right-hand-side kernel on two copies of
the field, sampled sites against the oracle, and a solve for the norms.

Bar 1e-12 in the norm and per sampled site, as for FP64 operators elsewhere."""
import numpy as np
import pytest

from oracle import wilson as W
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd import wilson_eo as WE
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from paper_2303_08609_amd.solve import cg
from tests._helpers import AP, cached_gauge, rel_err, sample_sites, site_rel_max

pytestmark = pytest.mark.gpu


# (34, 32, 24, 24): 4 strips of 6 planes, 3264 sites = 12.75 workgroups, a multiple of 64
# (32, 22, 40, 12): 8 strips of 5 planes, 1760 sites = 6.875 workgroups, no multiple of 64
# (32, 22, 40, 10): too few t slices, lexicographic
@pytest.mark.parametrize("dims", [(34, 32, 24, 24), (32, 22, 40, 12), (32, 22, 40, 10)],
                         ids=lambda d: "x".join(map(str, d)))
def test_strips(dims):
    print(f"hop strips {dims}", flush=True)
    fmt, lat, ph = Format("f64", "f64", 12), Lattice(dims, 0.12, AP), np.array(AP, dtype=np.complex128)
    u, psi = cached_gauge(dims, 0.4, 1900), inputs.gen_spinor_half(dims, 1901)
    u_d, psi_d = lat.pack_gauge(to_device(u), fmt), to_device(psi)
    x_d = lat.pack_spinor(psi_d, fmt)
    x2 = lat.pack_spinor(psi_d.unsqueeze(0).repeat(2, 1, 1, 1, 1, 1, 1), fmt)
    sites = sample_sites(dims, 24, 13)
    for dag in (False, True):
        got = lat.unpack_spinor(lat.apply(u_d, x_d, fmt, dagger=dag), fmt).cpu().numpy()
        ref = lat.unpack_spinor(lat.apply(u_d, x2, fmt, dagger=dag, nrhs=2), fmt, nrhs=2).cpu().numpy()
        assert rel_err(got, ref[0]) <= 1e-12 and rel_err(got, ref[1]) <= 1e-12, dag
        want = W.apply_m_at_sites(u, psi, 0.12, ph, sites, dagger=dag)
        assert site_rel_max(got.reshape(-1, 4, 3)[sites], want) <= 1e-12, dag
    x, info = cg(lat, fmt, u_d, x_d, tol=1e-8, maxiter=500)
    assert info["status"] == WE.WEO_OK, info
    r = lat.unpack_spinor(lat.apply(u_d, x, fmt), fmt).cpu().numpy() - psi
    assert np.linalg.norm(r) <= 2e-8 * np.linalg.norm(psi)
