"""Canonical copies and snapshots move whole 16-byte vectors, and their tails
singly: every value arrives, and nothing beside it is written."""
import pytest
import torch

from paper_1703_04594_amd.lbm import Lattice

from _util import G, TAU, TB, TT, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# rows: below a vector, whole vectors, one to three over, a segment of one and
# of several chunks, arrays on either side of the non-temporal bound
@pytest.mark.parametrize("lx,ly", [(7, 7), (9, 8), (11, 130), (5 + 8, 1029), (64, 2051), (7, 4097), (1000, 1501)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("layout", ["columns", "planes"])
def test_canonical_copies_and_snapshots(lx, ly, precision, layout):
    say(f"copies {lx}x{ly} {precision} {layout}")
    dt = torch.float64 if precision == "fp64" else torch.float32
    lat = Lattice(lx, ly, TAU, G, TB, TT, precision=precision, layout=layout, device=DEV)
    n = 37 * lx * ly
    f = (torch.arange(n, device=DEV, dtype=torch.float64) % 16777216).to(dt).reshape(37, lx, ly)
    guard = torch.full((n + 64,), -7.0, dtype=dt, device=DEV)
    # a source and a destination that start one element off a 16-byte boundary
    src = torch.empty(n + 1, dtype=dt, device=DEV)[1:].reshape(37, lx, ly)
    src.copy_(f)
    lat.set_pops(src)
    assert torch.equal(lat.get_pops(), f)
    dst = guard[33:33 + n].reshape(37, lx, ly)
    lat._run("get_pops", lat.L.lbm_get_pops, dst.data_ptr())
    assert torch.equal(dst, f)
    assert bool((guard[:33] == -7.0).all()) and bool((guard[33 + n:] == -7.0).all())
    # a snapshot on a 256-byte boundary, and one at an odd address
    raw = torch.full((lat.state_bytes + 1024,), 0x5A, dtype=torch.uint8, device=DEV)
    for off in (256, 3):
        st = raw[off:off + lat.state_bytes]
        lat.get_state(st)
        assert bool((raw[:off] == 0x5A).all()) and bool((raw[off + lat.state_bytes:] == 0x5A).all())
        other = Lattice(lx, ly, TAU, G, TB, TT, precision=precision, layout=layout, device=DEV)
        other.set_state(st)
        assert torch.equal(other.get_pops(), f)
        assert torch.equal(other.get_state(), lat.get_state())
        raw.fill_(0x5A)
