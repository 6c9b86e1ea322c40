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


# both sides of the streaming bound of the read-outs and initial states, and of
# the totals' row condition
@pytest.mark.parametrize("lx,ly", [(7, 7), (33, 70), (1024, 1024), (1024, 1030)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_initial_states_and_read_outs(lx, ly, precision):
    """The wall densities that init leaves are those of a state set from its
    populations (bitwise: one sum in one order), and macros and totals are the
    moments of the populations: sums of 37 terms in FP64 differ by at most
    37 ulp between summation orders, totals of N sites by sqrt(N) of those."""
    say(f"initial states {lx}x{ly} {precision}")
    import oracle
    lat, other = (Lattice(lx, ly, TAU, G, TB, TT, precision=precision, device=DEV) for _ in range(2))
    g = torch.Generator(device=DEV).manual_seed(3)
    P = torch.rand((lx, ly), generator=g, device=DEV, dtype=torch.float64)
    lat.init_rt(P)
    for _ in range(2):
        other.set_pops(lat.get_pops())
        assert torch.equal(lat.get_state(), other.get_state())
        lat.init(1.0 + 0.1 * P, 0.02 * P, -0.01 * P, 1.0 + 0.05 * P)
    f = lat.get_pops().double()
    if precision == "fp32":
        f = f + torch.tensor(oracle.weights(), device=DEV)[:, None, None]
    ex, ey = oracle.velocity_table()
    c = oracle.scale_c()
    xi = [torch.tensor([c * float(v) for v in e], dtype=torch.float64, device=DEV)[:, None, None] for e in (ex, ey)]
    rho = f.sum(0)
    j = [(x * f).sum(0) for x in xi]
    en = ((xi[0] ** 2 + xi[1] ** 2) * f).sum(0)
    T = (en / rho - (j[0] ** 2 + j[1] ** 2) / rho ** 2) / 2
    tol = 37 * 2.3e-16 * 10          # sum of |terms| over the sum: at most 10 for the energy
    for a, b in zip(lat.macros(), (rho, j[0] / rho, j[1] / rho, T)):
        assert float((a - b).abs().max()) <= tol
    tot = torch.stack([rho.sum(), j[0].sum(), j[1].sum(), en.sum()])
    assert bool(((lat.conservation() - tot).abs() <= tol * lx * ly).all())


# segments of 4 to 9 waves of vectors: chunks of fewer waves than a block has,
# the last wave full, with one vector, with one element
@pytest.mark.parametrize("rows", [256, 257, 320, 321, 384, 449, 512, 513, 576])
@pytest.mark.parametrize("tail", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_copies_of_long_segments(rows, tail, precision):
    lx, ly = 9, rows * (2 if precision == "fp64" else 4) - tail
    say(f"long segments {lx}x{ly} {precision}")
    dt = torch.float64 if precision == "fp64" else torch.float32
    lat = Lattice(lx, ly, TAU, G, TB, TT, precision=precision, device=DEV)
    n = 37 * lx * ly
    f = torch.arange(n, device=DEV, dtype=torch.float64).to(dt).reshape(37, lx, ly)
    lat.set_pops(f)
    guard = torch.full((n + 64,), -7.0, dtype=dt, device=DEV)
    lat._run("get_pops", lat.L.lbm_get_pops, guard[32:32 + n].data_ptr())
    assert torch.equal(guard[32:32 + n], f.reshape(-1))
    assert bool((guard[:32] == -7.0).all()) and bool((guard[32 + n:] == -7.0).all())


# without walls a snapshot is the buffer alone: the runtime's copy below the
# streaming bound, the kernel beyond it, and either at an odd address
@pytest.mark.parametrize("lx,ly", [(7, 7), (40, 33), (700, 700)])
@pytest.mark.parametrize("off", [256, 3])
def test_snapshots_without_walls(lx, ly, off):
    say(f"snapshots without walls {lx}x{ly} +{off}")
    a, b = (Lattice(lx, ly, TAU, G, TB, TT, precision="fp64", ybc="periodic", device=DEV) for _ in range(2))
    f = torch.arange(37 * lx * ly, device=DEV, dtype=torch.float64).reshape(37, lx, ly)
    a.set_pops(f)
    raw = torch.full((a.state_bytes + 1024,), 0x5A, dtype=torch.uint8, device=DEV)
    st = raw[off:off + a.state_bytes]
    a.get_state(st)
    assert bool((raw[:off] == 0x5A).all()) and bool((raw[off + a.state_bytes:] == 0x5A).all())
    b.set_state(st)
    assert torch.equal(b.get_pops(), f)
