"""What tuning costs the first call of a key: z strips of any lattice do not
multiply the shapes that are timed."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

_CHILD = r"""
import torch
from paper_2303_08609_amd.ops import Format, Lattice
lat, fmt = Lattice((12, 12, 12, 24), 0.12, (1, 1, 1, -1)), Format("f16", "f16", 12)
u, x = (torch.zeros(n, dtype=torch.uint8, device="cuda") for n in (lat.gauge_bytes(fmt), lat.spinor_bytes(fmt, 12)))
lat.hop(u, x, fmt, 1, nrhs=12)
torch.cuda.synchronize()
"""


def test_shapes_timed_for_one_key():
    """12 FP16/12 fields on planes that fill no whole workgroups, the key with
    the most kernels: 95 shapes without strips (1 single-field, 24 with links in
    registers, 30 in LDS, 40 groups of fields) and 3 strip heights of the 8
    fastest."""
    print("shapes timed for one key", flush=True)
    env = dict(os.environ, WEO_TUNE_VERBOSE="1")
    for k in ("WEO_TUNE", "WILSON_EO_TUNE_CACHE"):
        env.pop(k, None)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    p = subprocess.run([sys.executable, "-c", _CHILD], env=env, cwd=root, capture_output=True, text=True, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    timed = [ln for ln in p.stderr.splitlines() if ln.startswith("[weo tune] fmt")]
    finals = [ln for ln in p.stderr.splitlines() if ln.startswith("[weo tune] final")]
    print(f"  {len(timed)} shapes, {len(finals)} again", flush=True)
    assert len(finals) == 4
    assert any(" bz 0 " not in ln for ln in timed)
    assert len(timed) <= 95 + 3 * 8
