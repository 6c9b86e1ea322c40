"""The FP64 step and the reverse step with FP64 lambda run 64- or 256-thread
blocks by the number of rows.  Sizes around the rule's edges and the blocks',
walls included, against the CPU oracle: the bars of the forward and the
adjoint tests for one step of each (rounding of FP64 sums)."""
import pytest
import torch

from oracle.ref_torch import TorchD2Q37
from paper_1703_04594_amd import inputs
from paper_1703_04594_amd.lbm import Lattice

from _util import TB, TT, TAU, W, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
WT = torch.tensor(W, dtype=torch.float64)[:, None, None]


@pytest.mark.parametrize("ly", [7, 64, 65, 192, 193, 256, 257, 333])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
def test_steps_match_the_oracle(ly, ybc):
    lx, g = 9, -1e-3
    say(f"block sizes {lx}x{ly} {ybc}")
    f0 = WT * (1 + 0.05 * torch.tensor(inputs.population_noise(lx, ly, 31)))
    lam2 = torch.tensor(inputs.population_noise(lx, ly, 32))
    lat = Lattice(lx, ly, TAU, g, TB, TT, precision="fp64", ybc=ybc, step="fused", adjoint="fp64", device=DEV)
    lat.set_pops(f0.to(DEV))
    states = [lat.get_state()]
    lat.step(1)
    f1 = lat.get_pops().cpu()
    states.append(lat.get_state())
    lat.set_lambda(lam2.to(DEV))
    dtau = torch.zeros((), dtype=torch.float64, device=DEV)
    for s in reversed(states):      # the second one gathers the first one's result
        lat.adjoint_step(s, dtau)
    lam0 = lat.get_lambda().cpu()

    m = TorchD2Q37(lx, ly, g, TB, TT, walls=(ybc == "walls"))
    f = f0.clone().requires_grad_(True)
    tau = torch.tensor(TAU, dtype=torch.float64, requires_grad=True)
    s1 = m.step(f, tau)
    (m.step(s1, tau) * lam2).sum().backward()
    e_f = float(((f1 - s1.detach()).abs() / WT).max())
    e_l = float((lam0 - f.grad).abs().max() / f.grad.abs().max())
    e_t = abs(float(dtau) - float(tau.grad)) / abs(float(tau.grad))
    say(f"  f {e_f:.2e}  lambda {e_l:.2e}  dtau {e_t:.2e}")
    assert e_f <= 1e-13 and e_l <= 1e-12 and e_t <= 1e-12


# working sets (two buffers) below, inside and beyond the range that takes cached
# loads and stores: bitwise the fused step, which evaluates the same expressions
@pytest.mark.parametrize("lx,ly", [(200, 250), (301, 333), (512, 400), (1000, 900)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("ybc,layout,xmode", [("walls", "columns", "wrap"), ("periodic", "planes", "halo")])
def test_split_steps_equal_fused_ones(lx, ly, precision, ybc, layout, xmode):
    say(f"split and fused {lx}x{ly} {precision} {ybc} {layout} {xmode}")
    P = torch.tensor(inputs.rt_perturbation(lx, ly, 7), device=DEV)
    out = []
    for step in ("split", "fused"):
        lat = Lattice(lx, ly, TAU, -1e-3, TB, TT, precision=precision, ybc=ybc, layout=layout, xmode=xmode, step=step,
                      device=DEV)
        lat.init_rt(P)
        for _ in range(3):
            lat.step(1)
        out.append(lat.get_pops())
    assert torch.equal(out[0], out[1])
