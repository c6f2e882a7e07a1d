"""The link gradient and su(3) force kernel where its workgroups end: 8 and
240 half sites (partly filled wavefronts), whole workgroups, every storage
format, both output precisions, accumulation, complex phases; against the
oracle on the rounded fields.

Bar: FP64 arithmetic on the stored values, about 60 operations per entry of
matrices of order 10: 1e-13; an output in FP32 adds its rounding, 6e-8 (twice
where it is accumulated): 2e-7.
"""
import numpy as np
import pytest
import torch

from oracle import force as F
from oracle.lattice import half_to_full
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd import wilson_eo as W
from paper_2303_08609_amd.ops import Format, Lattice, _ptr, _stream, to_device
from tests._helpers import ROUND, link_as_stored, rel_err

pytestmark = pytest.mark.gpu

CPX = tuple(np.exp(1j * np.array([0.4, -1.1, 2.0, 2.9])))
FORMATS = [("f64", "f64", 18), ("f64", "f64", 12), ("f32", "f32", 18), ("f32", "f32", 12), ("f16", "f16", 12),
           ("bf16", "f16", 18)]


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 2, 10), (8, 4, 4, 4)], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("fmt_t", FORMATS, ids=lambda f: f"{f[0]}-{f[1]}-{f[2]}")
def test_force_edges(fmt_t, dims):
    sp, lp, reals = fmt_t
    print(f"force dims={dims} fmt={fmt_t}", flush=True)
    fmt, lat = Format(*fmt_t), Lattice(dims, 0.125, CPX)
    # values the formats hold exactly; Lambda_e, Lambda_o, R_e, R_o
    u = ROUND[lp](inputs.gen_gauge(dims, 0.5, 1600))
    f = [ROUND[sp](inputs.gen_spinor_half(dims, 1601 + k)) for k in range(4)]
    d = [lat.pack_spinor(to_device(x), fmt) for x in f]
    u_d = lat.pack_gauge(to_device(u), fmt)
    u_o = link_as_stored(u, lp, reals)
    full = [half_to_full(f[2 * k], 0, dims) + half_to_full(f[2 * k + 1], 1, dims) for k in (0, 1)]
    grad = F.link_grad_bilinear(u_o, full[0], full[1], -0.3, np.array(CPX))
    for flags, want in ((0, grad), (W.WEO_FORCE_PROJECT, F.force_from_grad(u_o, grad))):
        for dt, prec, bar in ((torch.complex128, W.WEO_F64, 1e-13), (torch.complex64, W.WEO_F32, 2e-7)):
            for acc in (0, W.WEO_FORCE_ACCUMULATE):
                base = torch.full(lat.gauge_shape(), 0.5 - 0.25j, dtype=dt, device="cuda")
                out = base.clone()
                W.check(W.wilson_eo_force(lat.c, fmt.c, _ptr(u_d), *(_ptr(x) for x in d), -0.3, flags | acc, _ptr(out),
                                          prec, _stream()), "wilson_eo_force")
                w = want + (base.cpu().numpy() if acc else 0)
                assert rel_err(out.cpu().numpy().astype(np.complex128), w) <= bar, (flags, dt, acc)
