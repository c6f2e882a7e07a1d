"""What wilson_apply keeps for backward: no more than its inputs on lattices
whose links are large, and the same gradients whether the packed fields were
kept, packed again, or came back converted by a saved-tensor hook; a link
gradient alone, and the adjoint.

Bars: 1e-12 relative in the norm against the oracle in FP64; the hook rounds u
and psi to FP32, 2e-6 as for FP32 gradients elsewhere."""
import numpy as np
import pytest
import torch

from oracle import force as F
from oracle import wilson as W
from paper_2303_08609_amd import autograd as A
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd.ops import Lattice, to_device
from tests._helpers import AP, rel_err

pytestmark = pytest.mark.gpu

DIMS, KAPPA, PH = (4, 6, 2, 8), 0.125, np.array(AP, dtype=np.complex128)


def _small():
    u, psi, eta = inputs.gen_gauge(DIMS, 0.5, 501), *(inputs.gen_spinor_half(DIMS, s) for s in (502, 503))
    return u, psi, eta, Lattice(DIMS, KAPPA, AP)


def _normal(shape, gen, scale=1.0):
    return torch.view_as_complex(scale * torch.randn(shape + (2,), generator=gen, device="cuda", dtype=torch.float64))


def test_large_links_are_not_kept():
    print("graph memory 32^4", flush=True)
    lat, gen = Lattice((32, 32, 32, 32), 0.12, AP), torch.Generator(device="cuda").manual_seed(7)
    u = _normal(lat.gauge_shape(), gen, 0.4).requires_grad_(True)
    psi = _normal(lat.half_shape(), gen).requires_grad_(True)
    A.wilson_apply(u.detach(), psi.detach(), lat)       # the library is loaded
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    out = A.wilson_apply(u, psi, lat)
    torch.cuda.synchronize()
    grown = torch.cuda.memory_allocated() - before
    print(f"  {grown / 2**20:.0f} MiB for an output of {out.numel() * 16 / 2**20:.0f}", flush=True)
    assert grown <= 1.01 * out.numel() * 16


def test_kept_and_packed_again_give_the_same(monkeypatch):
    print("kept / packed again", flush=True)
    u, psi, eta, lat = _small()
    grads = []
    for limit in (A.KEEP_LINK_BYTES, 0):
        monkeypatch.setattr(A, "KEEP_LINK_BYTES", limit)
        ut, pt = to_device(u).requires_grad_(True), to_device(psi).requires_grad_(True)
        grads.append(torch.autograd.grad(A.wilson_apply(ut, pt, lat), (ut, pt), to_device(eta)))
    for a, b in zip(*grads):
        assert torch.equal(a, b)
    assert rel_err(grads[1][0].cpu().numpy(), F.link_grad_l1(u, psi, eta, KAPPA, PH)) <= 1e-12
    assert rel_err(grads[1][1].cpu().numpy(), F.grad_psi_l1(u, eta, KAPPA, PH)) <= 1e-12


def test_saved_tensor_hook_that_converts():
    print("saved-tensor hook", flush=True)
    u, psi, eta, lat = _small()
    ut, pt = to_device(u).requires_grad_(True), to_device(psi).requires_grad_(True)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.to(torch.complex64), lambda t: t.to(torch.complex128)):
        out = A.wilson_apply(ut, pt, lat)
    g_u, g_psi = torch.autograd.grad(out, (ut, pt), to_device(eta))
    assert rel_err(g_u.cpu().numpy(), F.link_grad_l1(u, psi, eta, KAPPA, PH)) <= 2e-6
    assert rel_err(g_psi.cpu().numpy(), F.grad_psi_l1(u, eta, KAPPA, PH)) <= 2e-6


@pytest.mark.parametrize("limit", [A.KEEP_LINK_BYTES, 0])
def test_links_alone_and_adjoint(limit, monkeypatch):
    print(f"links alone, adjoint, limit {limit}", flush=True)
    monkeypatch.setattr(A, "KEEP_LINK_BYTES", limit)
    u, psi, eta, lat = _small()
    ut, pt, et = to_device(u).requires_grad_(True), to_device(psi), to_device(eta)
    g_u, = torch.autograd.grad(A.wilson_apply(ut, pt, lat), (ut,), et)
    assert rel_err(g_u.cpu().numpy(), F.link_grad_l1(u, psi, eta, KAPPA, PH)) <= 1e-12
    pt.requires_grad_(True)
    out = A.wilson_apply(ut.detach(), pt, lat, True)
    assert rel_err(out.detach().cpu().numpy(), W.apply_m(u, psi, KAPPA, PH, dagger=True)) <= 1e-12
    g_psi, = torch.autograd.grad(out, (pt,), et)
    assert rel_err(g_psi.cpu().numpy(), W.apply_m(u, eta, KAPPA, PH)) <= 1e-12
    with pytest.raises(NotImplementedError):
        torch.autograd.grad(A.wilson_apply(ut, pt, lat, True), (ut,), et)
