"""lbm_create does not clear the adjoint state: no result depends on what the
caller's memory held.  The workspace is the test's own, filled before the
context is created in it."""
import ctypes

import pytest
import torch

from paper_1703_04594_amd.lbm import Lattice, workspace_bytes

from _util import G, TAU, TB, TT, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def lattice_over(byte, lx, ly, **kw):
    """A lattice whose context was created in memory full of that byte (0xFF: NaN)."""
    lat = Lattice(lx, ly, TAU, G, TB, TT, device=DEV, step="fused", **kw)
    lat.close()
    lat.workspace.fill_(byte)
    h = ctypes.c_void_p()
    st = lat.L.lbm_create(ctypes.byref(lat.p), ctypes.c_void_p(lat._ws_ptr), workspace_bytes(lat.p),
                          ctypes.c_void_p(lat.stream.cuda_stream), ctypes.byref(h))
    assert st == 0
    lat.h = h
    return lat


# 200x333: more elements than one round of the kernel's blocks
@pytest.mark.parametrize("lx,ly", [(7, 7), (40, 33), (200, 333)])
@pytest.mark.parametrize("lam", ["fp64", "fp32"])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
def test_lambda_before_a_seed_is_zero(lx, ly, lam, ybc):
    say(f"lambda before a seed {lx}x{ly} {lam} {ybc}")
    lat = lattice_over(0xFF, lx, ly, precision="fp32", ybc=ybc, adjoint=lam)
    assert torch.equal(lat.get_lambda(), torch.zeros((37, lx, ly), dtype=torch.float64, device=DEV))
