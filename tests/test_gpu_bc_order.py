"""lbm_bc reads the state before the current one, whatever calls stand between:
it is refused where there is no such state, and equals the same call after
single steps, bitwise, where there is."""
import pytest
import torch

from paper_1703_04594_amd import inputs
from paper_1703_04594_amd.lbm import Lattice, LBMError

from _util import G, TAU, TB, TT, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def lattice(lx, ly, **kw):
    lat = Lattice(lx, ly, TAU, G, TB, TT, device=DEV, step="fused", **kw)
    lat.init_rt(torch.tensor(inputs.rt_perturbation(lx, ly, 5), device=DEV))
    return lat


# n = 2: one pass, straight into the snapshot; 1 and 3: a single step, one more pass
@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("source", ["snapshot", "lattice"])
@pytest.mark.parametrize("target", ["snapshot", "lattice"])
def test_bc_is_refused_after_an_advance(n, source, target):
    say(f"bc after advance_state n={n} {source} {target}")
    lat = lattice(40, 33, precision="fp64")
    s0, out = lat.get_state(), lat.new_state()
    lat.step(4)
    lat.advance_state(s0 if source == "snapshot" else None, out if target == "snapshot" else None, n)
    with pytest.raises(LBMError):
        lat.bc()
    lat.propagate()
    lat.bc()


# A replay advances the state without the host: eager steps and replays of both
# kinds (single steps, passes of two) before the bc, an even number each, so that
# the graph's buffers are those it was captured with.  "c4": capture of 4 steps,
# "r": its replay, "4": eager steps.
ORDERS = [["2", "c4", "r", "2", "r"], ["2", "c4", "r", "2"], ["2", "c2", "r", "4", "r"], ["2", "c2", "4", "r", "4"],
          ["4", "c2"], ["2", "c4"], ["2", "c6", "4", "r", "r", "8"]]


@pytest.mark.parametrize("order", ORDERS, ids="-".join)
@pytest.mark.parametrize("lx,ly,precision", [(40, 33, "fp64"), (129, 257, "fp32"), (901, 1458, "fp32")])
def test_bc_among_replays_equals_single_steps(lx, ly, precision, order):
    say(f"bc among replays {lx}x{ly} {precision} {order}")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a, b = (lattice(lx, ly, precision=precision) for _ in range(2))
    graph, n = None, 0
    for op in order:
        if op[0] == "c":
            graph, n = torch.cuda.CUDAGraph(), int(op[1:])
            s.synchronize()
            with torch.cuda.graph(graph, stream=s):
                a.step(n)
            continue
        with torch.cuda.stream(s):
            if op == "r":
                graph.replay()
            else:
                a.step(int(op))
            for _ in range(n if op == "r" else int(op)):
                b.step(1)
    with torch.cuda.stream(s):
        a.bc()
        b.bc()
        after_bc = [x.get_pops() for x in (a, b)]
        a.step(1)
        b.step(1)
        after_step = [x.get_pops() for x in (a, b)]
        a.bc()
        b.bc()
        last = [x.get_pops() for x in (a, b)]
    s.synchronize()
    assert torch.equal(*after_bc) and torch.equal(*after_step) and torch.equal(*last)


# propagate, bc and collide one by one after passes of two steps and replays of
# them, and captured themselves: "p" the three kernels, "cp" a capture of them twice
PIECES = [["4", "p", "p", "4", "p"], ["2", "c4", "p", "p", "r", "p"], ["2", "c4", "r", "p"], ["4", "cp", "p"],
          ["2", "cp", "4", "r", "p", "p", "r"], ["2", "cp", "r", "4", "p"]]


@pytest.mark.parametrize("order", PIECES, ids="-".join)
@pytest.mark.parametrize("lx,ly,precision", [(40, 33, "fp64"), (129, 257, "fp32"), (901, 1458, "fp32")])
def test_kernels_one_by_one_equal_steps(lx, ly, precision, order):
    say(f"kernels one by one {lx}x{ly} {precision} {order}")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a, b = (lattice(lx, ly, precision=precision) for _ in range(2))

    def pieces(times):
        for _ in range(times):
            a.propagate()
            a.bc()
            a.collide()

    graph, n = None, 0
    for op in order:
        if op[0] == "c":
            graph, n = torch.cuda.CUDAGraph(), 2 if op == "cp" else int(op[1:])
            s.synchronize()
            with torch.cuda.graph(graph, stream=s):
                pieces(2) if op == "cp" else a.step(n)
            continue
        with torch.cuda.stream(s):
            if op == "r":
                graph.replay()
            elif op == "p":
                pieces(1)
            else:
                a.step(int(op))
            for _ in range(n if op == "r" else 1 if op == "p" else int(op)):
                b.step(1)
            got, want = a.get_pops(), b.get_pops()
        s.synchronize()
        assert torch.equal(got, want), op
