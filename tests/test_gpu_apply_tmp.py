"""wilson_eo_apply leaves H_oe in (H_oe^dag in) in tmp, bit for bit what
wilson_eo_hop writes for one field and to rounding for several (their two
launches may be tuned to different kernels): on both sides of the
small-lattice limit, in strips, for several fields.

Bars for several fields as in the other operator tests, 1e-12 / 1e-6 / 2e-3."""
import pytest
import torch

from paper_2303_08609_amd.ops import Format, Lattice
from tests._helpers import AP

pytestmark = pytest.mark.gpu

REAL = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}
TOL = {"f64": 1e-12, "f32": 1e-6, "f16": 2e-3}


@pytest.mark.parametrize("dims, sp, nrhs", [((6, 4, 2, 10), "f64", 1), ((18, 14, 18, 18), "f32", 1),
                                            ((34, 32, 24, 24), "f64", 1), ((6, 4, 2, 10), "f32", 5),
                                            ((18, 14, 18, 18), "f16", 3)])
def test_apply_leaves_the_odd_half(dims, sp, nrhs):
    print(f"tmp of apply {dims} {sp} nrhs={nrhs}", flush=True)
    lat, fmt, gen = Lattice(dims, 0.12, AP), Format(sp, None, 12), torch.Generator(device="cuda").manual_seed(5)
    size = REAL[sp].itemsize
    u, x = ((s * torch.randn(n // size, generator=gen, device="cuda")).to(REAL[sp]).view(torch.uint8)
            for s, n in ((0.4, lat.gauge_bytes(fmt)), (1.0, lat.spinor_bytes(fmt, nrhs))))
    for dag in (False, True):
        tmp = torch.zeros_like(x)
        lat.apply(u, x, fmt, dagger=dag, nrhs=nrhs, tmp=tmp)
        hop = lat.hop(u, x, fmt, 1, dagger=dag, nrhs=nrhs)
        if nrhs == 1:
            assert torch.equal(tmp, hop)
        a, b = (v.view(REAL[sp]).double() for v in (tmp, hop))
        assert b.norm() > 0 and (a - b).norm() <= TOL[sp] * b.norm()
