"""Workloads of the even-odd Wilson operator whose speed is tracked.

A case is one call, or one short fixed sequence of calls, as a lattice program
makes them: operator applications (the inner loop of every solve), the
clover-type operator, the autograd derivative and the su(3) force of molecular
dynamics, the conversion of a new gauge configuration, one device's share of a
split hop, the Schwarz preconditioner, and one whole mixed-precision solve.
Lattices run from 4^4 to 48^3x96; right-hand sides from 1 to 12 (the twelve
spin-colour sources of a propagator).

``listed`` names the tracked cases, ``draw`` gives further ones of the same
ranges, ``prepare`` builds what the program holds before the call, ``run`` is
one pass, ``work`` its unavoidable bytes and floating-point operations, and
``exact`` the same result in FP64 from plain torch.
"""
import math

import torch

from paper_2303_08609_amd import autograd as A
from paper_2303_08609_amd.ops import Format, Lattice
from paper_2303_08609_amd.solve import cg

BC = (1, 1, 1, -1)              # periodic in space, antiperiodic in time
REAL = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
TORCH = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SAP = dict(block=(4, 4, 4, 4), ncy=4, nmr=4)


def _case(kind, dims, kappa=0.126, eps=0.5, spinor="f32", reals=18, nrhs=1, dagger=False, option=""):
    lx, ly, lz, lt = dims
    return dict(kind=kind, lx=lx, ly=ly, lz=lz, lt=lt, kappa=kappa, eps=eps, spinor=spinor, reals=reals, nrhs=nrhs,
                dagger=bool(dagger), option=option)


def listed():
    return [
        # the smallest lattice used in earnest (dense cross-checks, tests of a
        # program): two hops of 128 sites each, all launch latency
        dict(_case("apply", (4, 4, 4, 4), 0.125, 0.3, "f64"), name="apply_f64_4x4x4x4"),
        # the headline: one M apply on the standard volume
        dict(_case("apply", (32, 32, 32, 64)), name="apply_f32_32x32x32x64"),
        # the inner operator of the mixed solve on the large volume
        dict(_case("apply", (48, 48, 48, 96), 0.1265, 0.7, "f16", 12, 1, True), name="apply_f16_48x48x48x96"),
        # the twelve propagator sources in one call, the inner operator of the
        # batched mixed solve
        dict(_case("apply", (32, 32, 32, 64), spinor="f16", reals=12, nrhs=12), name="apply_f16_12rhs_32x32x32x64"),
        # a few sources on a lattice of no convenient size, FP64 residual operator
        dict(_case("apply", (20, 12, 28, 36), spinor="f64", reals=12, nrhs=5), name="apply_f64_5rhs_20x12x28x36"),
        # the clover-type operator, one source
        dict(_case("clover", (32, 32, 32, 64)), name="clover_f32_32x32x32x64"),
        # the clover-type operator on the twelve sources
        dict(_case("clover", (16, 16, 16, 32), spinor="f16", reals=12, nrhs=12), name="clover_f16_12rhs_16x16x16x32"),
        # forward and backward of M psi in FP64: gradients of both inputs
        dict(_case("grad", (16, 16, 16, 32), 0.125, 0.5, "f64"), name="grad_f64_16x16x16x32"),
        # a new configuration: links for the FP64 and the FP16 operators, the
        # twelve sources in, the twelve solutions out
        dict(_case("load", (24, 24, 24, 48), spinor="f16", reals=12, nrhs=12), name="load_f16_24x24x24x48"),
        # one device's share of 32^3x64 cut along t into 8 slabs
        dict(_case("split", (32, 32, 32, 8), option="t"), name="split_t_f32_32x32x32x8"),
        # one application of the Schwarz preconditioner (4^4 blocks, 4 cycles
        # of 4 steps) inside flexible GCR
        dict(_case("sap", (32, 32, 32, 64)), name="sap_f32_32x32x32x64"),
        # twelve sources to 1e-10: FP64 defect correction around FP16 BiCGStab
        dict(_case("solve", (16, 16, 16, 32), 0.126, 0.5, "f16", 12, 12), name="solve_f16_12rhs_16x16x16x32"),
    ]


def _dims(rng, lo, hi, step=2):
    """Four even extents (multiples of step), volume log-uniform in [lo, hi]."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    side = (v / 2) ** 0.25
    d = [max(step, step * int(round(side * rng.uniform(0.6, 1.5) / step))) for _ in range(3)]
    t = int(round(v / (d[0] * d[1] * d[2]) / step)) * step
    d.append(min(96, max(step, t)))
    while d[0] * d[1] * d[2] * d[3] > 1.2 * hi:
        d[3] = max(step, step * int(d[3] / 2 / step))
        if d[3] == step:
            d[0] = max(step, d[0] - step)
    return tuple(d)


def draw(rng):
    kind = rng.choices(["apply", "clover", "grad", "force", "load", "split", "sap", "solve"],
                       [6, 3, 2, 2, 2, 2, 2, 2])[0]
    std = 32 ** 3 * 64
    spinor, reals = rng.choice([("f64", 18), ("f64", 12), ("f32", 18), ("f32", 12), ("f16", 18), ("f16", 12),
                                ("bf16", 12)])
    kappa, eps = round(rng.uniform(0.118, 0.127), 4), round(rng.uniform(0.3, 0.7), 2)
    dag = rng.random() < 0.5
    if kind == "apply":
        nrhs = rng.choice([1, 1, 1, 2, 3, 4, 6, 8, 12])
        return _case(kind, _dims(rng, 256, std / max(1, nrhs / 4)), kappa, eps, spinor, reals, nrhs, dag)
    if kind == "clover":
        nrhs = rng.choice([1, 1, 2, 3, 4, 6, 12])
        return _case(kind, _dims(rng, 256, std / max(1, nrhs / 2)), kappa, eps, spinor, reals, nrhs, dag)
    if kind == "grad":
        return _case(kind, _dims(rng, 256, 24 ** 3 * 48), kappa, eps, rng.choice(["f64", "f32"]))
    if kind == "force":
        return _case(kind, _dims(rng, 256, 24 ** 3 * 48), kappa, eps, rng.choice(["f64", "f32"]))
    if kind == "load":
        return _case(kind, _dims(rng, 256, 24 ** 3 * 48), kappa, eps, spinor, reals, rng.choice([1, 2, 4, 12]),
                     option=rng.choice(["", "", "clover"]))
    if kind == "split":
        return _case(kind, _dims(rng, 256, std / 4), kappa, eps, spinor, reals, rng.choice([1, 1, 4]), dag,
                     rng.choice(["t", "zt", "xyzt"]))
    if kind == "sap":
        nrhs = rng.choice([1, 1, 2])
        return _case(kind, _dims(rng, 4096, std / 1.2 / nrhs, 8), kappa, eps, "f32", rng.choice([18, 12]), nrhs)
    spinor = rng.choice(["f16", "f32", "bf16"])
    return _case(kind, _dims(rng, 256, 16 ** 3 * (14 if spinor == "f32" else 26)), kappa, eps, spinor, 12,
                 rng.choice([1, 2, 4, 12]))


# ---- inputs -----------------------------------------------------------------
def _dims_of(c):
    return c["lx"], c["ly"], c["lz"], c["lt"]


def _fmt(c):
    return Format(c["spinor"], None, c["reals"])


def _gen(seed, role):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 16 + role)


def _normal(shape, gen):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=gen, dtype=torch.float64, device="cuda"))


def _links(c, seed):
    """Near-unit SU(3) links [4][Lt][Lz][Ly][Lx][3][3]: the exponential of
    i eps H to second order, rows re-orthonormalised, row 2 = conj(row0 x row1)."""
    lx, ly, lz, lt = _dims_of(c)
    gen = _gen(seed, 1)
    out = torch.empty((4, lt, lz, ly, lx, 3, 3), dtype=torch.complex128, device="cuda")
    one = torch.eye(3, dtype=torch.complex128, device="cuda")
    for mu in range(4):
        a = _normal((lt, lz, ly, lx, 3, 3), gen)
        h = 0.5 * c["eps"] * (a + a.mH)
        h2 = (h.unsqueeze(-1) * h.unsqueeze(-3)).sum(-2)
        w = one + 1j * h - 0.5 * h2
        r0 = w[..., 0, :] / w[..., 0, :].abs().square().sum(-1, keepdim=True).sqrt()
        r1 = w[..., 1, :] - (r0.conj() * w[..., 1, :]).sum(-1, keepdim=True) * r0
        r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
        out[mu, ..., 0, :] = r0
        out[mu, ..., 1, :] = r1
        out[mu, ..., 2, :] = _row2(r0, r1)
    return out


def _row2(r0, r1):
    i, j = [1, 2, 0], [2, 0, 1]
    return (r0[..., i] * r1[..., j] - r0[..., j] * r1[..., i]).conj()


def _half(c, seed, role, nrhs=1):
    """Gaussian one-parity fields [nrhs][Lt][Lz][Ly][Lx/2][4][3]."""
    lx, ly, lz, lt = _dims_of(c)
    return _normal((nrhs, lt, lz, ly, lx // 2, 4, 3), _gen(seed, role))


def _blocks(c, seed):
    """Clover-type site blocks near one, [Lt][Lz][Ly][Lx][2][6][6]."""
    lx, ly, lz, lt = _dims_of(c)
    g = _normal((lt, lz, ly, lx, 2, 6, 6), _gen(seed, 6))
    return torch.eye(6, dtype=torch.complex128, device="cuda") + 0.2 / math.sqrt(6.0) * 0.5 * (g + g.mH)


def _canon(c):
    return torch.complex128 if c["spinor"] == "f64" else torch.complex64


class _State:
    pass


def _split_dirs(c):
    return tuple("xyzt".index(d) for d in c["option"])


def prepare(case, seed):
    c, s = case, _State()
    s.c = c
    s.lat = Lattice(_dims_of(c), c["kappa"], BC)
    s.fmt = _fmt(c)
    n, kind = c["nrhs"], c["kind"]
    u = _links(c, seed)
    if kind in ("grad", "force"):
        dt = _canon(c)
        s.u, s.psi = u.to(dt), _half(c, seed, 2)[0].to(dt)
        s.eta = _half(c, seed, 3)[0].to(dt)
        if kind == "grad":
            s.u.requires_grad_(True)
            s.psi.requires_grad_(True)
        return s
    if kind == "load":
        # the configuration and sources as read from disk, the packed
        # solutions to be written out, and the program's own packed buffers
        s.u, s.b = u, _half(c, seed, 2, n)
        s.f64 = Format("f64", "f64", 12)
        s.u64, s.uop = s.lat.new_gauge(s.f64), s.lat.new_gauge(s.fmt)
        s.bp = s.lat.new_spinor(s.f64, n)
        s.x = s.lat.pack_spinor(_half(c, seed, 3, n), s.f64)
        if c["option"] == "clover":
            s.blocks = _blocks(c, seed)
            s.cp = torch.empty(s.lat.clover_bytes(s.fmt), dtype=torch.uint8, device="cuda")
        return s
    s.u = s.lat.pack_gauge(u, s.fmt)
    if kind == "sap":
        eta = [s.lat.pack_spinor(_half(c, seed, 2 + p, n), s.fmt).view(n, -1) for p in (0, 1)]
        s.eta = torch.cat(eta, dim=1).reshape(-1)       # per source: even half, odd half
        s.out = s.lat.new_spinor(s.fmt, 2 * n)
        return s
    if kind == "solve":
        s.f64 = Format("f64", "f64", 12)
        s.u64 = s.lat.pack_gauge(u, s.f64)
        s.b = s.lat.pack_spinor(_half(c, seed, 2, n), s.f64)
        s.out = s.lat.new_spinor(s.f64, n)
        return s
    s.x = s.lat.pack_spinor(_half(c, seed, 2, n), s.fmt)
    s.out = s.lat.new_spinor(s.fmt, n)
    if kind == "split":
        s.dirs = _split_dirs(c)
        s.bulk = s.lat.open_dirs(s.dirs)
        s.faces = {mu: [torch.empty(s.lat.face_bytes(s.fmt, n, mu), dtype=torch.uint8, device="cuda")
                        for _ in range(2)] for mu in s.dirs}
        return s
    s.tmp = s.lat.new_spinor(s.fmt, n)
    if kind == "clover":
        s.clv = s.lat.pack_clover(_blocks(c, seed), s.fmt, invert=True)
    return s


# ---- one pass ---------------------------------------------------------------
def run(s):
    c, lat, fmt, n = s.c, s.lat, s.fmt, s.c["nrhs"]
    kind, dag = c["kind"], c["dagger"]
    if kind == "apply":
        return lat.apply(s.u, s.x, fmt, dagger=dag, nrhs=n, out=s.out, tmp=s.tmp).view(TORCH[c["spinor"]])
    if kind == "clover":
        return lat.clover_apply(s.u, s.clv, s.x, fmt, dagger=dag, nrhs=n, out=s.out,
                                tmp=s.tmp).view(TORCH[c["spinor"]])
    if kind == "grad":
        out = A.wilson_apply(s.u, s.psi, lat)
        g_u, g_psi = torch.autograd.grad(out, (s.u, s.psi), s.eta)
        return out.detach(), g_u, g_psi
    if kind == "force":
        return A.link_force_l1(s.u, s.psi, s.eta, lat)
    if kind == "load":
        lat.pack_gauge(s.u, s.f64, out=s.u64)
        lat.pack_gauge(s.u, fmt, out=s.uop)
        lat.pack_spinor(s.b, s.f64, out=s.bp)
        x = lat.unpack_spinor(s.x, s.f64, n, dtype=torch.complex128)
        link = torch.float16 if c["spinor"] in ("f16", "bf16") else TORCH[c["spinor"]]
        res = [s.u64.view(torch.float64), s.uop.view(link), s.bp.view(torch.float64), x]
        if c["option"] == "clover":
            res.append(lat.pack_clover(s.blocks, fmt, invert=True, out=s.cp).view(link))
        return res
    if kind == "split":
        # every face goes to the block itself: one device standing for a row of them
        for mu in s.dirs:
            lat.face_pack(s.u, s.x, fmt, 1, dagger=dag, nrhs=n, lo=s.faces[mu][0], hi=s.faces[mu][1], mu=mu)
        s.bulk.hop(s.u, s.x, fmt, 1, dagger=dag, nrhs=n, out=s.out)
        for mu in s.dirs:
            lat.face_unpack(s.u, s.faces[mu][1], s.faces[mu][0], s.out, fmt, 1, dagger=dag, phase_lo=BC[mu],
                            phase_hi=BC[mu], nrhs=n, mu=mu)
        return s.out.view(TORCH[c["spinor"]])
    if kind == "sap":
        return lat.sap(s.u, s.eta, fmt, nrhs=n, out=s.out, **SAP).view(torch.float32)
    inner_tol = 1e-5 if c["spinor"] == "f32" else 1e-3
    x, _ = cg(lat, s.f64, s.u64, s.b, nrhs=n, tol=1e-10, inner=fmt, u_inner=s.u, inner_tol=inner_tol, out=s.out,
              method="bicgstab")
    return x.view(torch.float64)


# ---- what a pass cannot do without --------------------------------------------
def work(case):
    """A hop reads every link once and its fields once: the second hop of an
    apply needs all of the first one's output, so the links count per hop."""
    c = case
    lx, ly, lz, lt = _dims_of(c)
    v, n, kind = lx * ly * lz * lt, c["nrhs"], c["kind"]
    vh = v // 2
    sb = 24 * REAL[c["spinor"]]
    lr = 2 if c["spinor"] == "bf16" else REAL[c["spinor"]]
    links = 4 * v * c["reals"] * lr
    hop = links + 2 * n * vh * sb
    flop = 1320 * vh * n
    clv = v * 2 * 36 * lr
    if kind == "apply":
        return {"bytes": 2 * hop + n * vh * sb, "flops": 2 * flop}
    if kind == "clover":
        return {"bytes": 2 * hop + n * vh * sb + clv, "flops": 2 * flop + v * n * 2 * 6 * 6 * 8}
    if kind == "grad":
        # M psi, M^dag g, the two hops for the odd halves and the outer products;
        # links in and gradient out once each
        return {"bytes": 2 * links + 7 * vh * sb, "flops": 6 * flop + 4 * v * 2 * 2 * 9 * 8}
    if kind == "force":
        return {"bytes": 2 * links + 2 * vh * sb, "flops": 2 * flop + 4 * v * (2 * 2 * 9 * 8 + 27 * 8)}
    if kind == "load":
        b = 2 * 4 * v * 18 * 8 // 2 + 4 * v * 12 * 8 + links + 4 * n * vh * 24 * 8
        if c["option"] == "clover":
            b += v * 2 * 72 * 8 + clv
        return {"bytes": b, "flops": v * 2 * 6 ** 3 * 8 if c["option"] == "clover" else 0}
    if kind == "split":
        return {"bytes": hop, "flops": flop}
    if kind == "sap":
        # per sweep of one colour: the links of its blocks, its residual and
        # solution in and out; one block operator per step on half the sites
        sweeps = 2 * SAP["ncy"]
        return {"bytes": sweeps * (links // 2 + 4 * n * vh * sb), "flops": sweeps * SAP["nmr"] * flop}
    # two FP64 residuals and 24 inner operator applications per source set:
    # what a residual of 1e-10 takes at these couplings
    res = 2 * (2 * (4 * v * 12 * 8 + 2 * n * vh * 192) + n * vh * 192)
    return {"bytes": res + 24 * (2 * hop + n * vh * sb), "flops": 26 * 2 * flop}


# ---- the same in FP64 with plain torch ------------------------------------------
# gamma_mu has one entry per row: (gamma_mu psi)_s = G[mu][s] psi_{PERM[mu][s]}
_PERM = ([3, 2, 1, 0], [3, 2, 1, 0], [2, 3, 0, 1], [0, 1, 2, 3])
_G = ([-1j, -1j, 1j, 1j], [-1, 1, 1, -1], [-1j, 1j, 1j, -1j], [1, 1, -1, -1])


def _parity_sel(c, par):
    lx, ly, lz, lt = _dims_of(c)
    t, z, y = (torch.arange(k, device="cuda") for k in (lt, lz, ly))
    s = (t[:, None, None] + z[None, :, None] + y[None, None, :] + par) & 1
    return s[:, :, :, None, None, None]


def _full(c, half, par):
    """[..., Lx/2, 4, 3] of one parity -> the full lattice, zero elsewhere."""
    s = _parity_sel(c, par).to(torch.float64)
    f = torch.stack([half * (1 - s), half * s], dim=-3)
    lx = c["lx"]
    return f.reshape(half.shape[:-3] + (lx, 4, 3))


def _take(c, full, par):
    s = _parity_sel(c, par) == 1
    f = full.reshape(full.shape[:-3] + (c["lx"] // 2, 2, 4, 3))
    return torch.where(s, f[..., 1, :, :], f[..., 0, :, :])


def _gam(mu, psi):
    g = torch.tensor(_G[mu], dtype=torch.complex128, device=psi.device)
    return psi[..., _PERM[mu], :] * g[:, None]


def _mul(u, psi):
    return sum(u[..., None, :, b] * psi[..., b, None] for b in range(3))


def _shift(psi, mu, sign, lead):
    """psi at x + sign mu-hat with the boundary phase."""
    ax = lead + 3 - mu
    out = torch.roll(psi, -sign, dims=ax)
    if BC[mu] != 1:
        n = out.shape[ax]
        ph = torch.ones(n, dtype=torch.float64, device=psi.device)
        ph[n - 1 if sign > 0 else 0] = BC[mu]
        out = out * ph.reshape([n if k == ax else 1 for k in range(out.dim())])
    return out


def _hop(u, psi, dagger=False, keep=None):
    """H psi on the full lattice (leading source axes allowed); keep[mu][0 / 1]
    masks the forward / backward terms."""
    lead = psi.dim() - 6
    sg = -1 if dagger else 1
    out = torch.zeros_like(psi)
    for mu in range(4):
        f = _mul(u[mu], _shift(psi, mu, 1, lead))
        f = f - sg * _gam(mu, f)
        out = out + (f if keep is None else f * keep[mu][0])
        b = _shift(_mul(u[mu].mH, psi), mu, -1, lead)
        b = b + sg * _gam(mu, b)
        out = out + (b if keep is None else b * keep[mu][1])
    return out


def _apply(c, u, x, dagger=False):
    t = _hop(u, _full(c, x, 0), dagger)
    return x - c["kappa"] ** 2 * _take(c, _hop(u, t, dagger), 0)


def _round(x, prec):
    """Canonical complex values as stored in precision prec, in FP64."""
    if prec == "f64":
        return x
    r = torch.view_as_real(x).float()
    if prec != "f32":
        r = r.to(TORCH[prec])
    return torch.view_as_complex(r.double().contiguous())


def _stored_links(c, u, prec=None, reals=None):
    prec = prec or c["spinor"]
    v = _round(u, "f16" if prec == "bf16" else prec)
    if (reals or c["reals"]) == 12:
        v = torch.cat([v[..., :2, :], _row2(v[..., 0, :], v[..., 1, :]).unsqueeze(-2)], dim=-2)
    return v


def _planes(x, nbytes):
    """[n][k][vh][records] complex -> the packed order: per record field,
    planes of 16 bytes, then the rest."""
    r = torch.view_as_real(x.contiguous()).reshape(x.shape[:-1] + (-1,))     # [..., vh, reals]
    k = 16 // nbytes
    m = r.shape[-1] // k * k
    a = r[..., :m].reshape(r.shape[:-1] + (m // k, k)).transpose(-3, -2)
    a = a.reshape(r.shape[:-2] + (-1,))
    b = r[..., m:].reshape(r.shape[:-2] + (-1,))
    return torch.cat([a, b], dim=-1).reshape(-1)


def _packed(c, x, prec=None):
    """[n][Lt][Lz][Ly][Lx/2][4][3] -> packed values."""
    return _planes(x.reshape(x.shape[0], -1, 12), REAL[prec or c["spinor"]])


def _parities(c, full, tail):
    """[..., Lt, Lz, Ly, Lx, tail...] -> [..., 2, vh, prod(tail)] by parity."""
    lx, ly, lz, lt = _dims_of(c)
    k = math.prod(tail)
    f = full.reshape(-1, lt, lz, ly, lx // 2, 2, k)
    res = []
    for par in (0, 1):
        s = _parity_sel(c, par).reshape(lt, lz, ly, 1, 1) == 1
        res.append(torch.where(s, f[..., 1, :], f[..., 0, :]).reshape(f.shape[0], -1, k))
    return torch.stack(res, dim=1)


def _inverse(b):
    n = b.numel() // 36
    return torch.linalg.inv(b.reshape(n, 6, 6).cpu()).to(b.device).reshape(b.shape)


def _site(inv, psi):
    """Inverse blocks on a full-lattice spinor (gamma5 eigenbasis)."""
    up, dn = psi[..., :2, :].flatten(-2), psi[..., 2:, :].flatten(-2)
    a, b = up + dn, up - dn
    a = sum(inv[..., 0, :, k] * a[..., k, None] for k in range(6))
    b = sum(inv[..., 1, :, k] * b[..., k, None] for k in range(6))
    return torch.cat([0.5 * (a + b), 0.5 * (a - b)], dim=-1).reshape(psi.shape)


def _clover(c, u, inv, x, dagger):
    f = _full(c, x, 0)
    if not dagger:
        f = _hop(u, _site(inv, _hop(u, f)))
        return x - c["kappa"] ** 2 * _take(c, _site(inv, f), 0)
    f = _hop(u, _site(inv, _hop(u, _site(inv, f), True)), True)
    return x - c["kappa"] ** 2 * _take(c, f, 0)


def _gradient(c, u, psi, eta):
    """Gradient with respect to the links of Re <eta, M psi>."""
    lam, r = _full(c, eta, 0), _full(c, psi, 0)
    lam = lam + _hop(u, lam, True)
    r = r + _hop(u, r)
    out = torch.empty_like(u)
    for mu in range(4):
        w = lam - _gam(mu, lam)
        v = _shift(r, mu, 1, 0)
        g = sum(w[..., s, :, None] * v[..., s, None, :].conj() for s in range(4))
        wp = _shift(lam + _gam(mu, lam), mu, 1, 0)
        g = g + sum(r[..., s, :, None] * wp[..., s, None, :].conj() for s in range(4))
        out[mu] = -c["kappa"] ** 2 * g
    return out


def _block_sum(v, lead):
    """Sums over 4^4 blocks, spread over their sites again."""
    s, n = v, v.shape
    dims = n[lead:lead + 4]
    s = s.reshape(n[:lead] + tuple(k for d in dims for k in (d // 4, 4)))
    ax = [lead + 1 + 2 * k for k in range(4)]
    return s.sum(dim=ax, keepdim=True).expand(n[:lead] + tuple(k for d in dims for k in (d // 4, 4))).reshape(n)


def _sap(c, u, eta):
    lx, ly, lz, lt = _dims_of(c)
    pos = [torch.arange(k, device="cuda") for k in (lt, lz, ly, lx)]
    col = sum((p // 4).reshape([-1 if k == i else 1 for k in range(4)]) for i, p in enumerate(pos)) & 1
    keep = []
    for mu in range(4):
        p = pos[3 - mu]
        whole = p.numel() == 4
        shape = [-1 if k == 3 - mu else 1 for k in range(4)] + [1, 1]
        f = torch.ones_like(p) if whole else (p % 4 != 3)
        b = torch.ones_like(p) if whole else (p % 4 != 0)
        keep.append([m.reshape(shape).to(torch.float64) for m in (f, b)])
    psi, rho = torch.zeros_like(eta), eta
    lead = eta.dim() - 6
    for _ in range(SAP["ncy"]):
        for colour in (0, 1):
            on = (col == colour)[..., None, None].to(torch.float64)
            r, e = rho * on, torch.zeros_like(eta)
            for _ in range(SAP["nmr"]):
                q = (r - c["kappa"] * _hop(u, r, keep=keep)) * on
                num = _block_sum((q.conj() * r).sum((-2, -1)), lead)
                den = _block_sum(q.abs().square().sum((-2, -1)), lead)
                al = torch.where(den > 0, num / den.clamp_min(1e-300), 0 * num)[..., None, None]
                e, r = e + al * r, r - al * q
            psi = psi + e
            rho = rho - (e - c["kappa"] * _hop(u, e))
    return psi


def _solve(c, u, b):
    """M x = b by CG on the normal equations to 1e-13."""
    def dot(p, q):
        return (p.conj() * q).flatten(1).sum(1).real[(slice(None),) + (None,) * 6]
    x, s = torch.zeros_like(b), b.clone()
    r = _apply(c, u, s, True)
    p, gam, bb = r, dot(r, r), dot(b, b)
    for _ in range(400):
        q = _apply(c, u, p)
        al = gam / dot(q, q).clamp_min(1e-300)
        x, s = x + al * p, s - al * q
        if bool((dot(s, s) <= 1e-26 * bb).all()):
            return x
        r = _apply(c, u, s, True)
        new = dot(r, r)
        p, gam = r + (new / gam) * p, new
    return None


def exact(case, seed):
    c, n, kind = case, case["nrhs"], case["kind"]
    u = _links(c, seed)
    prec = c["spinor"]
    if kind in ("grad", "force"):
        if prec == "f32":
            u = _round(u, "f32")
        psi, eta = (_round(_half(c, seed, k)[0], prec) for k in (2, 3))
        g = _gradient(c, u, psi, eta)
        if kind == "grad":
            return _apply(c, u, psi), g, _apply(c, u, eta, True)
        y = 1j * sum(u[..., :, k, None] * g.conj()[..., None, :, k] for k in range(3))
        h = 0.5 * (y + y.mH)
        tr = torch.diagonal(h, dim1=-2, dim2=-1).sum(-1)[..., None, None] / 3.0
        return h - tr * torch.eye(3, dtype=torch.complex128, device="cuda")
    if kind == "load":
        rows = c["reals"] // 6
        lp = "f16" if prec == "bf16" else prec
        res = [_planes(_parities(c, u[..., :2, :], (2, 3)), 8),
               _planes(_parities(c, _round(u, lp)[..., :rows, :], (rows, 3)), REAL[lp]),
               _packed(c, _half(c, seed, 2, n), "f64"), _half(c, seed, 3, n).reshape(Lattice(
                   _dims_of(c), c["kappa"], BC).half_shape(n if n > 1 else None))]
        if c["option"] == "clover":
            inv = _inverse(_blocks(c, seed))
            lx, ly, lz, lt = _dims_of(c)
            d = torch.diagonal(inv, dim1=-2, dim2=-1).real.contiguous()
            i, j = torch.tril_indices(6, 6, -1)
            rec = torch.cat([torch.view_as_complex(d.reshape(d.shape[:-1] + (3, 2))), inv[..., i, j]], dim=-1)
            p = _parities(c, rec.movedim(4, 0).contiguous(), (18,)).transpose(0, 1).contiguous()
            res.append(_planes(_round(p, lp), REAL[lp]))
        return res
    us = _stored_links(c, u)
    if kind == "sap":
        halves = [_round(_half(c, seed, 2 + p, n), "f32") for p in (0, 1)]
        psi = _sap(c, us, _full(c, halves[0], 0) + _full(c, halves[1], 1))
        out = torch.stack([_take(c, psi, 0), _take(c, psi, 1)], dim=1)
        return _planes(out.reshape(2 * n, -1, 12), 4)
    if kind == "solve":
        x = _solve(c, _stored_links(c, u, "f64", 12), _half(c, seed, 2, n))
        return None if x is None else _packed(c, x, "f64")
    x = _round(_half(c, seed, 2, n), prec)
    res = []
    inv = _round(_inverse(_blocks(c, seed)), "f16" if prec == "bf16" else prec) if kind == "clover" else None
    for r in range(n):          # one source at a time: the large cases stay small in memory
        if kind == "apply":
            y = _apply(c, us, x[r], c["dagger"])
        elif kind == "clover":
            y = _clover(c, us, inv, x[r], c["dagger"])
        else:
            y = _take(c, _hop(us, _full(c, x[r], 0), c["dagger"]), 1)
        res.append(_planes(y.reshape(1, -1, 12), REAL[prec]))
    return torch.cat(res)
