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
