"""Canonical <-> packed conversion where a wavefront's 64 records end: fewer
records than lanes, a ragged last wavefront, wavefronts that cross from one
right-hand side to the next; both canonical precisions, every storage format.
Conversions round to nearest even (FP64 through FP32 to 16 bits), so the
values are compared bit by bit."""
import pytest
import torch

from paper_2303_08609_amd.ops import Format, Lattice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spinor", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("dims, nrhs", [((2, 2, 2, 2), 1), ((4, 2, 2, 2), 3), ((6, 2, 4, 2), 5), ((4, 4, 4, 2), 2),
                                        ((10, 6, 2, 6), 16)], ids=lambda v: str(v))
def test_spinor_round_trip(spinor, dims, nrhs):
    print(f"round trip {spinor} {dims} nrhs={nrhs}", flush=True)
    lat, fmt = Lattice(dims, 0.12), Format(spinor)
    gen = torch.Generator().manual_seed(17)
    for dt, real in ((torch.complex128, torch.float64), (torch.complex64, torch.float32)):
        x = torch.view_as_complex(torch.randn(lat.half_shape(nrhs) + (2,), generator=gen, dtype=real)).cuda()
        x = x if nrhs > 1 else x[0].contiguous()
        store = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[spinor]
        r = torch.view_as_real(x)
        want = (r.to(store) if spinor in ("f64", "f32") else r.float().to(store)).double()
        p = lat.pack_spinor(x, fmt)
        for out, f in ((torch.complex128, torch.float64), (torch.complex64, torch.float32)):
            got = torch.view_as_real(lat.unpack_spinor(p, fmt, nrhs=nrhs, scale=0.5, dtype=out))
            assert got.shape == want.shape
            assert torch.equal(got, (0.5 * want).to(f))
