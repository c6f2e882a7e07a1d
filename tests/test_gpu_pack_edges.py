"""Packed -> canonical conversion where a wavefront's 64 records end: fewer
records than lanes, a ragged last wavefront, wavefronts that cross from one
right-hand side to the next; both canonical precisions, every storage format.
Every stored value is exact in either canonical precision (FP64 values rounded
once to FP32), so the values are compared bit by bit."""
import pytest
import torch

from paper_2303_08609_amd.ops import Format, Lattice

pytestmark = pytest.mark.gpu

STORE = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


@pytest.mark.parametrize("spinor", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("dims, nrhs", [((2, 2, 2, 2), 1), ((4, 2, 2, 2), 3), ((6, 2, 4, 2), 5), ((4, 4, 4, 2), 2),
                                        ((10, 6, 2, 6), 16)], ids=lambda v: str(v))
def test_unpack(spinor, dims, nrhs):
    print(f"unpack {spinor} {dims} nrhs={nrhs}", flush=True)
    lat, fmt = Lattice(dims, 0.12), Format(spinor)
    v = torch.randn(nrhs, lat.vh, 24, generator=torch.Generator().manual_seed(17), dtype=torch.float64)
    v = v.to(STORE[spinor]).cuda()
    k = 16 // v.element_size()                      # planes of 16 bytes per site
    packed = v.reshape(nrhs, lat.vh, 24 // k, k).transpose(1, 2).contiguous().reshape(-1).view(torch.uint8)
    assert packed.numel() == lat.spinor_bytes(fmt, nrhs)
    for out, f in ((torch.complex128, torch.float64), (torch.complex64, torch.float32)):
        got = torch.view_as_real(lat.unpack_spinor(packed, fmt, nrhs=nrhs, scale=0.5, dtype=out))
        assert torch.equal(got.reshape(nrhs, lat.vh, 24), (0.5 * v.double()).to(f))
