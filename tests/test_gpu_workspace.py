"""lbm_create does not clear the adjoint state: no result depends on what the
caller's memory held.  The workspace is the test's own, filled before the
context is created in it."""
import ctypes

import pytest
import torch

from paper_1703_04594_amd import inputs
from paper_1703_04594_amd.lbm import Lattice, LBMError, workspace_bytes

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


@pytest.mark.parametrize("lx,ly", [(7, 7), (40, 33)])
@pytest.mark.parametrize("lam", ["fp64", "fp32"])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_reverse_steps_in_memory_that_held_nan(precision, ybc, lam, lx, ly):
    """The padding of the adjoint state still holds the NaN that the test wrote;
    the sweep equals one in memory that held zeros, bitwise."""
    say(f"reverse steps over NaN {lx}x{ly} {precision} {ybc} {lam}")
    gT = torch.tensor(inputs.uniform_field(lx, ly, 4, -1, 1), device=DEV)
    P = torch.tensor(inputs.rt_perturbation(lx, ly, 5), device=DEV)
    out = []
    for byte in (0, 0xFF):
        lat = lattice_over(byte, lx, ly, precision=precision, ybc=ybc, adjoint=lam)
        lat.init_rt(P)
        states = [lat.get_state()]
        for _ in range(2):
            lat.step(1)
            states.append(lat.get_state())
        lat.step(1)
        lat.seed_temperature(gT)
        dtau = torch.zeros((), dtype=torch.float64, device=DEV)
        for s in reversed(states):
            lat.adjoint_step(s, dtau)
        lat.seed_temperature(gT)
        for s in reversed(states):
            lat.adjoint_step(s, None)
        lat.take_dtau(dtau)
        out.append((lat.get_lambda(), lat.adjoint_init_rt(P), dtau))
        if byte:
            assert bool((lat.workspace.view(torch.int32) == -1).any())
    for a, b in zip(*out):
        assert torch.isfinite(b).all() and torch.equal(a, b)


# a snapshot given twice, and two that overlap
def test_overlapping_snapshots_are_refused():
    lat = Lattice(40, 33, TAU, G, TB, TT, precision="fp64", step="fused", device=DEV)
    n = lat.state_bytes
    mem = torch.zeros(2 * n + 512, dtype=torch.uint8, device=DEV)
    off = -mem.data_ptr() % 256
    a, b = mem[off:off + n], mem[off + n - 256:off + 2 * n - 256]
    for src, dst in ((a, a), (a, b), (b, a)):
        with pytest.raises(LBMError, match="overlap"):
            lat.advance_state(src, dst, 2)
        with pytest.raises(LBMError, match="overlap"):
            lat.step_state(src, dst)
    with pytest.raises(LBMError, match="n < 1"):
        lat.advance_state(None, None, 0)
