"""The multi right-hand-side kernels that take their links from LDS, where
they can go wrong: ragged last workgroups, fewer and more right-hand sides
than wavefronts, every format, clover blocks staged next to the links, the
packed FP16 form (reached through a tuning cache), phases 0 (open directions),
capture before anything is tuned.

Bars as in the other operator tests, per format: 1e-12 / 1e-6 / 2e-3 / 1e-2
relative in the norm against the FP64 oracle on the rounded inputs (about 300
operations per component at the arithmetic's rounding, and one rounding of
the stored output: 2^-11 and 2^-8 for FP16 and BF16, twice for an apply).
"""
import json
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from oracle import clover as CL
from oracle import wilson as W
from oracle.lattice import full_to_half
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd import wilson_eo as WE
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from tests._helpers import AP, ROUND, cached_gauge, link_as_stored, rel_err

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-6, "f16": 2e-3, "bf16": 1e-2}
FORMATS = [("f64", "f64", 18), ("f64", "f64", 12), ("f32", "f32", 18), ("f32", "f32", 12), ("f16", "f16", 18),
           ("f16", "f16", 12), ("bf16", "f16", 18), ("bf16", "f16", 12)]
CPX = tuple(np.exp(1j * np.array([0.4, -1.1, 2.0, 2.9])))
KAPPA = 0.124


@pytest.fixture(autouse=True)
def _reset_shape():
    yield
    WE.weo_set_mrhs_shape(0, 0, 0, 0, 0)


def _get(lat, fmt, x, nrhs):
    return lat.unpack_spinor(x, fmt, nrhs=nrhs).cpu().numpy()


@pytest.mark.parametrize("fmt_t", FORMATS, ids=lambda f: f"{f[0]}-{f[1]}-{f[2]}")
@pytest.mark.parametrize("nrhs", [2, 5, 13])
def test_clover_several_rhs(fmt_t, nrhs):
    dims = (10, 6, 4, 6)                    # 720 half sites: 16 in the last workgroup
    sp, lp, reals = fmt_t
    bc = CPX if nrhs == 5 else AP
    print(f"clover nrhs={nrhs} fmt={fmt_t}", flush=True)
    fmt, lat = Format(*fmt_t), Lattice(dims, KAPPA, bc)
    u = cached_gauge(dims, 0.5, 1500)
    blocks = inputs.gen_site_blocks(dims, 0.2, 1501)
    ainv = np.linalg.inv(CL.blocks_to_dirac(blocks))
    psi = inputs.gen_spinor_half(dims, 1502, nrhs=nrhs)
    y = inputs.gen_spinor_half(dims, 1503, nrhs=nrhs)
    u_d, x_d = lat.pack_gauge(to_device(u), fmt), lat.pack_spinor(to_device(psi), fmt)
    clv = lat.pack_clover(to_device(blocks), fmt)
    u_o, x_o, y_o = link_as_stored(u, lp, reals), ROUND[sp](psi), ROUND[sp](y)
    ai = [full_to_half(ainv, p) for p in (0, 1)]
    ph = np.array(bc, dtype=np.complex128)
    want = {d: [CL.apply_m_clover(u_o, x_o[r], KAPPA, ph, ai[0], ai[1], dagger=d) for r in range(nrhs)]
            for d in (False, True)}
    hop = [CL.apply_sites(ai[1], W.hop_eo(u_o, x_o[r], 0, ph)) for r in range(nrhs)]
    for shape in ((0, 0, 0, 0, 0), (-5, 2, 0, 0, 0), (-5, 12, 0, 0, 0), (-5, 3, 1, 2, 2), (1, 0, 0, 0, 0),
                  (-4, 256, 0, 0, 0)):
        assert WE.weo_set_mrhs_shape(*shape) == WE.WEO_OK
        for d in (False, True):
            got = _get(lat, fmt, lat.clover_apply(u_d, clv, x_d, fmt, dagger=d, nrhs=nrhs), nrhs)
            for r in range(nrhs):
                assert rel_err(got[r], want[d][r]) <= TOL[sp], (shape, d, r)
        y_d = lat.pack_spinor(to_device(y), fmt)
        got = _get(lat, fmt, lat.clover_hop(u_d, clv, x_d, fmt, 1, y=y_d, alpha=0.3, nrhs=nrhs, out=y_d), nrhs)
        for r in range(nrhs):
            assert rel_err(got[r], y_o[r] + 0.3 * hop[r]) <= TOL[sp], (shape, "in place", r)


@pytest.mark.parametrize("shape", [(-2, 64, 0, 0, 0), (-4, 256, 0, 0, 0), (-5, 4, 0, 0, 0), (0, 0, 0, 0, 0)])
def test_open_direction_several_rhs_fp16(shape):
    """A zero phase drops the hops across that edge for FP16 fields too."""
    dims, nrhs = (4, 4, 6, 8), 4
    print(f"open z, t; shape {shape}", flush=True)
    fmt, lat = Format("f16", "f16", 12), Lattice(dims, KAPPA, AP).open_dirs((2, 3))
    u, psi = inputs.gen_gauge(dims, 0.5, 1510), inputs.gen_spinor_half(dims, 1511, nrhs=nrhs)
    assert WE.weo_set_mrhs_shape(*shape) == WE.WEO_OK
    got = _get(lat, fmt, lat.hop(lat.pack_gauge(to_device(u), fmt), lat.pack_spinor(to_device(psi), fmt), fmt, 1,
                                 nrhs=nrhs), nrhs)
    u_o, x_o = link_as_stored(u, "f16", 12), ROUND["f16"](psi)
    for r in range(nrhs):
        assert rel_err(got[r], W.hop_eo(u_o, x_o[r], 0, np.array([1, 1, 0, 0], complex))) <= TOL["f16"], r


@pytest.mark.parametrize("dims", [(10, 6, 10, 4), (16, 8, 6, 4)], ids=["ragged", "aligned"])
@pytest.mark.parametrize("shape", [(-1, 256, 0, 4, 0), (-3, 64, 1, 3, 0), (3, 128, 0, 4, 0), (2, 64, 1, 4, 1),
                                   (-5, 4, 0, 4, 0), (-5, 3, 0, 7, 2)], ids=lambda s: ".".join(map(str, s)))
def test_strips_on_any_lattice(dims, shape):
    """z strips that do not divide Lz, on planes that fill no whole workgroups
    (30 half sites) and on planes of 64 (strips of 4 and then 2 planes, so
    256-site workgroups of the last strip are half filled): the hop with the
    axpy, and the norm partials through a solve."""
    from paper_2303_08609_amd.solve import cg
    nrhs, fmt = 5, Format("f32", "f32", 18)
    print(f"strips dims={dims} shape={shape}", flush=True)
    lat = Lattice(dims, KAPPA, AP)
    u = inputs.gen_gauge(dims, 0.5, 1540)
    psi, y = (inputs.gen_spinor_half(dims, 1541 + q, nrhs=nrhs) for q in (0, 1))
    u_d, x_d, y_d = (lat.pack_gauge(to_device(u), fmt), lat.pack_spinor(to_device(psi), fmt),
                     lat.pack_spinor(to_device(y), fmt))
    u_o, x_o, y_o = link_as_stored(u, "f32", 18), ROUND["f32"](psi), ROUND["f32"](y)
    ph = np.array(AP, dtype=np.complex128)
    assert WE.weo_set_mrhs_shape(*shape) == WE.WEO_OK
    got = _get(lat, fmt, lat.hop_axpy(u_d, x_d, y_d, fmt, 1, -0.3, nrhs=nrhs), nrhs)
    for r in range(nrhs):
        assert rel_err(got[r], y_o[r] - 0.3 * W.hop_eo(u_o, x_o[r], 0, ph)) <= TOL["f32"], r
    x_p, info = cg(lat, fmt, u_d, x_d, nrhs=nrhs, tol=1e-5, maxiter=2000)
    assert info["status"] == WE.WEO_OK, info
    x = _get(lat, fmt, x_p, nrhs)
    for r in range(nrhs):
        res = x_o[r] - W.apply_m(u_o, x[r], KAPPA, ph)
        assert np.linalg.norm(res) <= 3e-5 * np.linalg.norm(x_o[r]), r


def test_captured_before_tuning():
    """First calls of a key under capture record an untuned launch; replays
    equal the eager result."""
    dims, nrhs = (6, 4, 2, 10), 3
    print("capture before tuning", flush=True)
    fmt, lat = Format("f32", "f32", 18), Lattice(dims, KAPPA, AP)
    u_d = lat.pack_gauge(to_device(inputs.gen_gauge(dims, 0.5, 1520)), fmt)
    x = lat.pack_spinor(to_device(inputs.gen_spinor_half(dims, 1521, nrhs=nrhs)), fmt)
    clv = lat.pack_clover(to_device(inputs.gen_site_blocks(dims, 0.2, 1522)), fmt)
    out, out2, tmp = (lat.new_spinor(fmt, nrhs) for _ in range(3))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        lat.clover_apply(u_d, clv, x, fmt, nrhs=nrhs, out=out, tmp=tmp)
        lat.apply(u_d, x, fmt, nrhs=nrhs, out=out2, tmp=tmp)
    a = lat.clover_apply(u_d, clv, x, fmt, nrhs=nrhs).view(torch.float32)
    b = lat.apply(u_d, x, fmt, nrhs=nrhs).view(torch.float32)
    for _ in range(3):
        out.zero_()
        out2.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert (out.view(torch.float32) - a).norm() <= 1e-6 * a.norm()
        assert (out2.view(torch.float32) - b).norm() <= 1e-6 * b.norm()


_CHILD = r"""
import json, sys
import numpy as np
from oracle import wilson as W
from paper_2303_08609_amd import inputs
from paper_2303_08609_amd import wilson_eo as WE
from paper_2303_08609_amd.ops import Format, Lattice, to_device
from tests._helpers import ROUND, link_as_stored, rel_err
worst = 0.0
for k, (nrhs, bc) in enumerate(((12, (1, 1, 1, -1)), (5, tuple(np.exp(1j * np.array([0.4, -1.1, 2.0, 2.9])))))):
    for reals in (18, 12):
        dims = (6, 4, 4, 10)
        lat, fmt = Lattice(dims, 0.124, bc), Format("f16", "f16", reals)
        u = inputs.gen_gauge(dims, 0.5, 1530)
        psi, y = (inputs.gen_spinor_half(dims, 1531 + q, nrhs=nrhs) for q in (0, 1))
        ud, xd, yd = lat.pack_gauge(to_device(u), fmt), lat.pack_spinor(to_device(psi), fmt), \
            lat.pack_spinor(to_device(y), fmt)
        uo, xo, yo = link_as_stored(u, "f16", reals), ROUND["f16"](psi), ROUND["f16"](y)
        for dag in (False, True):
            h = lat.unpack_spinor(lat.hop(ud, xd, fmt, 1, dagger=dag, nrhs=nrhs), fmt, nrhs=nrhs).cpu().numpy()
            a = lat.unpack_spinor(lat.hop_axpy(ud, xd, yd, fmt, 1, -0.3, dagger=dag, nrhs=nrhs), fmt,
                                  nrhs=nrhs).cpu().numpy()
            for r in range(nrhs):
                w = W.hop_eo(uo, xo[r], 0, np.array(bc), dagger=dag)
                worst = max(worst, rel_err(h[r], w), rel_err(a[r], yo[r] - 0.3 * w))
rep = [json.loads(l) for l in WE.tuning_report().splitlines() if l.strip()]
print(json.dumps({"worst": worst, "nr": sorted({(e["nr"], e["sites"], e["split"]) for e in rep})}))
"""


@pytest.mark.parametrize("nr, waves, split", [(-7, 2, 0), (-7, 12, 0), (-7, 4, 6), (-8, 3, 0), (-8, 6, 0)])
def test_packed_fp16_lds_form(tmp_path, nr, waves, split):
    """Hop and axpy of the packed FP16 form in each of its shapes, chosen by a
    tuning cache with one entry per key (240 half sites: 48 in the last
    workgroup)."""
    path = tmp_path / "tune.txt"
    env = dict(os.environ, WILSON_EO_TUNE_CACHE=str(path))
    env.pop("WEO_TUNE", None)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

    def child():
        p = subprocess.run([sys.executable, "-c", _CHILD], env=env, cwd=root, capture_output=True, text=True,
                           timeout=120)
        assert p.returncode == 0, p.stderr[-2000:]
        return json.loads(p.stdout.strip().splitlines()[-1])

    print(f"packed FP16 LDS form nr={nr} waves={waves}: header", flush=True)
    assert child()["worst"] <= TOL["f16"]
    lines = path.read_text().splitlines()
    shaped = [" ".join(ln.split()[:7] + [str(nr), str(waves if int(ln.split()[5]) == 12 else min(waves, 6)), "0", "0",
                                         str(split if int(ln.split()[5]) == 12 else 0), "1.0"]) for ln in lines[1:]]
    path.write_text("\n".join(lines[:1] + shaped) + "\n")
    print(f"packed FP16 LDS form nr={nr} waves={waves}: forced", flush=True)
    res = child()
    assert {e[0] for e in res["nr"]} == {nr}, res
    assert res["worst"] <= TOL["f16"], res
