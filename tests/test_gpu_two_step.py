"""lbm_step takes fused steps two at a time in one pass over memory (tiles on
small lattices, a march along x on large ones), in groups of four steps.  Each
case compares step(n) with n calls of step(1), bitwise: both evaluate the same
expressions in the same order, so no tolerance applies.  (test_gpu_full_run.py
and test_gpu_random_configs.py hold step(n) to the oracle.)"""
import pytest
import torch

from paper_1703_04594_amd import inputs
from paper_1703_04594_amd.lbm import Lattice

from _util import G, TAU, TB, TT, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def pops(lx, ly, precision, seed):
    import oracle
    w = torch.tensor(oracle.weights(), device=DEV)[:, None, None]
    f = w * (1.0 + 0.02 * torch.tensor(inputs.population_noise(lx, ly, seed), device=DEV))
    return f if precision == "fp64" else (f - w).to(torch.float32)


def check(lx, ly, n, precision, ybc, layout="columns", xmode="wrap"):
    say(f"two steps per pass {lx}x{ly} n={n} {precision} {ybc} {layout} {xmode}")
    f = pops(lx, ly, precision, 5)
    a, b = (Lattice(lx, ly, TAU, G, TB, TT, precision=precision, ybc=ybc, step="fused", layout=layout, xmode=xmode,
                    device=DEV)
            for _ in range(2))
    a.set_pops(f)
    b.set_pops(f)
    a.step(n)
    for _ in range(n):
        b.step(1)
    assert torch.equal(a.get_pops(), b.get_pops())
    # the wall densities kept with the state, and those of the state before the
    # last step, which a further bc reads
    sa, sb = a.get_state(), b.get_state()
    c = Lattice(lx, ly, TAU, G, TB, TT, precision=precision, ybc=ybc, step="fused", layout=layout, xmode=xmode,
                    device=DEV)
    c.set_state(sa)
    b.set_state(sb)
    c.step(1)
    b.step(1)
    assert torch.equal(c.get_pops(), b.get_pops())
    if ybc == "walls":
        b.set_pops(f)
        for _ in range(n):
            b.step(1)
        a.bc()
        b.bc()
        a.step(1)
        b.step(1)
        assert torch.equal(a.get_pops(), b.get_pops())


# smallest lattice; tiles of 8x8, 8x16 and 16x16 with whole and ragged edges
# (one row or column over); lattices that a tile's ring wraps around
@pytest.mark.parametrize("lx,ly", [(7, 7), (8, 9), (17, 16), (40, 33), (128, 128), (129, 257), (230, 1030)])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_f32sums"])
def test_tiles(lx, ly, ybc, precision):
    check(lx, ly, 9, precision, ybc)


# the march: strips that end on a full strip, one row over, two rows over; a
# last segment of one column; the planes layout
@pytest.mark.parametrize("lx,ly", [(1024, 1120), (1200, 1121), (901, 1458), (2100, 1442)])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_f32sums"])
def test_march(lx, ly, ybc, precision):
    check(lx, ly, 5, precision, ybc, layout="planes" if lx == 901 else "columns")


# x halos: passes of two steps wrap the index, single steps copy the halos; a
# lattice for each of the forms
@pytest.mark.parametrize("lx,ly", [(7, 7), (129, 257), (901, 1458)])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_x_halos(lx, ly, ybc, precision):
    check(lx, ly, 5, precision, ybc, xmode="halo")


def test_march_largest():
    """4096x4096 FP64: a 5 GB buffer, beyond 32-bit offsets from its start."""
    check(4096, 4096, 4, "fp64", "walls")


@pytest.mark.parametrize("lx,ly", [(64, 64), (1024, 1024)])
def test_other_streams_and_rows_of_steps(lx, ly):
    """Two lattices stepped in turn on two streams, in uneven groups, end where
    each ends alone."""
    f = pops(lx, ly, "fp64", 6)
    alone = Lattice(lx, ly, TAU, G, TB, TT, precision="fp64", step="fused", device=DEV)
    alone.set_pops(f)
    for _ in range(21):
        alone.step(1)
    want = alone.get_pops()
    torch.cuda.synchronize()
    lats = []
    for _ in range(2):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            lat = Lattice(lx, ly, TAU, G, TB, TT, precision="fp64", step="fused", device=DEV)
            lat.set_pops(f)
        lats.append((s, lat))
    for n in (4, 1, 8, 2, 6):
        for s, lat in lats:
            with torch.cuda.stream(s):
                lat.step(n)
    for s, lat in lats:
        with torch.cuda.stream(s):
            got = lat.get_pops()
        s.synchronize()
        assert torch.equal(got, want)
