"""Hops of the clover operator on several right-hand sides take their launch
shape from a rule: no call is timed or waits for the stream, and on both sides
of every line of the rule the result is that of the single right-hand-side
kernel (packed random links, blocks and fields: only the kernels differ).

Bars as in the other operator tests, per format: 1e-12 / 1e-6 / 2e-3 / 1e-2
relative in the norm."""
import pytest
import torch

from paper_2303_08609_amd import wilson_eo as WE
from paper_2303_08609_amd.ops import Format, Lattice
from tests._helpers import AP

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-6, "f16": 2e-3, "bf16": 1e-2}
REAL = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
# half sites on both sides of 2^12, 2^13, 2^14, 2^15 and 2^17
LATTICES = [(8, 8, 8, 16), (18, 8, 8, 8), (10, 10, 16, 12), (16, 16, 16, 8), (18, 16, 16, 8), (16, 16, 16, 18),
            (32, 32, 32, 8), (34, 32, 32, 8)]


@pytest.fixture(autouse=True)
def _reset_shape():
    yield
    WE.weo_set_mrhs_shape(0, 0, 0, 0, 0)


def _rand(nbytes, dtype, scale, gen):
    n = nbytes // torch.empty(0, dtype=dtype).element_size()
    return (scale * torch.randn(n, generator=gen, device="cuda")).to(dtype).view(torch.uint8)


def _inputs(dims, sp, reals, nrhs):
    fmt, lat = Format(sp, None, reals), Lattice(dims, 0.12, AP)
    link = REAL["f16" if sp == "bf16" else sp]
    gen = torch.Generator(device="cuda").manual_seed(sum(dims) + nrhs)
    u = _rand(lat.gauge_bytes(fmt), link, 0.4, gen)
    clv = _rand(lat.clover_bytes(fmt), link, 0.3, gen)
    return fmt, lat, u, clv, _rand(lat.spinor_bytes(fmt, nrhs), REAL[sp], 1.0, gen)


@pytest.mark.parametrize("dagger", [False, True])
def test_clover_apply_does_not_wait(dagger):
    """Called behind queued work, the first apply of a lattice returns while
    that work still runs, and leaves nothing in the tuner."""
    print(f"clover apply behind queued work, dagger={dagger}", flush=True)
    nrhs = 3 if dagger else 4
    fmt, lat, u, clv, x = _inputs((12, 6, 8, 10), "f16", 12, nrhs)
    out, tmp = lat.new_spinor(fmt, nrhs), lat.new_spinor(fmt, nrhs)
    lat.clover_apply(u, clv, x, fmt, out=out, tmp=tmp)          # one field: the library is loaded
    a = torch.randn(8192, 8192, device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    before = WE.tuning_report()
    done = torch.cuda.Event()
    for _ in range(20):
        torch.mm(a, a, out=b)
    done.record()
    lat.clover_apply(u, clv, x, fmt, dagger=dagger, nrhs=nrhs, out=out, tmp=tmp)
    waited = done.query()
    torch.cuda.synchronize()
    assert not waited
    assert WE.tuning_report() == before


@pytest.mark.parametrize("sp, reals", [("f64", 12), ("f32", 18), ("f16", 12), ("bf16", 18)])
@pytest.mark.parametrize("dims", LATTICES, ids=lambda d: "x".join(map(str, d)))
def test_rule_matches_single_kernel(dims, sp, reals):
    for nrhs in (2, 3, 5, 7, 13):
        print(f"clover rule {dims} {sp}/{reals} nrhs={nrhs}", flush=True)
        fmt, lat, u, clv, x = _inputs(dims, sp, reals, nrhs)
        got = {}
        for shape in ((1, 0, 0, 0, 0), (0, 0, 0, 0, 0)):
            assert WE.weo_set_mrhs_shape(*shape) == WE.WEO_OK
            y = x.clone()
            got[shape[0]] = [lat.clover_apply(u, clv, x, fmt, dagger=d, nrhs=nrhs) for d in (False, True)] + \
                [lat.clover_hop(u, clv, x, fmt, 1, nrhs=nrhs),
                 lat.clover_hop(u, clv, x, fmt, 0, dagger=True, y=y, alpha=0.3, nrhs=nrhs, out=y)]
        for k, (one, rule) in enumerate(zip(got[1], got[0])):
            one, rule = (v.view(REAL[sp]).double() for v in (one, rule))
            assert torch.isfinite(one).all()
            assert (rule - one).norm() <= TOL[sp] * one.norm(), (nrhs, k)
