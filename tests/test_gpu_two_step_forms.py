"""Which form of the passes of two steps a lattice takes (on 256 CUs with 160 KB
of LDS), so that the tests that compare step(n) with single steps run what they
name, and the same comparison where a form begins or ends.  Bitwise: both
evaluate the same expressions in the same order."""
import pytest
import torch

from paper_1703_04594_amd import inputs
from paper_1703_04594_amd.lbm import Lattice

from _util import G, TAU, TB, TT, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def lattice(lx, ly, **kw):
    return Lattice(lx, ly, TAU, G, TB, TT, step="fused", device=DEV, **kw)


# the sizes of test_gpu_two_step.py, test_gpu_rollout_passes.py and test_gpu_bc_order.py
@pytest.mark.parametrize("form,sizes", [
    ("tile 8x8", [(7, 7), (8, 9), (17, 16), (40, 33), (64, 48), (64, 64), (128, 128)]),
    ("tile 16x16", [(129, 257), (230, 1030)]),
    ("march", [(901, 1458), (1024, 1024), (1024, 1120), (1200, 1121), (2100, 1442)])], ids=lambda v: v if isinstance(v, str) else "")
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_f32sums"])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
def test_forms_of_the_tested_sizes(form, sizes, precision, ybc):
    for lx, ly in sizes:
        for layout in ("columns", "planes"):
            for xmode in ("wrap", "halo"):
                assert lattice(lx, ly, precision=precision, ybc=ybc, layout=layout, xmode=xmode).two_step_form() == form
        assert Lattice(lx, ly, TAU, G, TB, TT, precision=precision, ybc=ybc, step="split",
                       device=DEV).two_step_form() == "none"


def test_forms_of_the_largest():
    assert lattice(2048, 4096, precision="fp64").two_step_form() == "march"
    assert lattice(2048, 4096, precision="fp32", layout="planes").two_step_form() == "march"
    # offsets between the populations of a site beyond 32 bits
    assert lattice(2048, 4096, precision="fp64", layout="planes").two_step_form() == "none"


# 8x16 tiles with ragged edges, tiles of FP64 and FP32 beyond the Infinity Cache,
# and FP32 beyond it where no form pays
@pytest.mark.parametrize("lx,ly,precision,form", [
    (129, 200, "fp64", "tile 8x16"), (129, 200, "fp32", "tile 8x16"), (129, 200, "fp32_f32sums", "tile 8x16"),
    (256, 128, "fp64", "tile 8x16"), (20000, 33, "fp64", "tile 16x16"), (3000, 300, "fp32", "tile 16x16"),
    (4096, 257, "fp32", "none")])
@pytest.mark.parametrize("ybc", ["walls", "periodic"])
def test_forms_equal_single_steps(lx, ly, precision, form, ybc):
    say(f"{form} {lx}x{ly} {precision} {ybc}")
    import oracle
    w = torch.tensor(oracle.weights(), device=DEV)[:, None, None]
    f = w * (1.0 + 0.02 * torch.tensor(inputs.population_noise(lx, ly, 5), device=DEV))
    f = f if precision == "fp64" else (f - w).to(torch.float32)
    a, b = (lattice(lx, ly, precision=precision, ybc=ybc) for _ in range(2))
    assert a.two_step_form() == form
    for lat in (a, b):
        lat.set_pops(f)
    a.step(5)
    for _ in range(5):
        b.step(1)
    assert torch.equal(a.get_pops(), b.get_pops())
    a.step(4)      # the wall densities that the passes leave
    for _ in range(4):
        b.step(1)
    a.bc()
    b.bc()
    assert torch.equal(a.get_pops(), b.get_pops())


# few columns: the tiles' rings are most of the work of a long lattice (FP32 with
# FP64 sums alone), on both sides of the shares and of the numbers of tiles
@pytest.mark.parametrize("lx,ly,form", [
    (17, 4096, "tile 16x16"), (17, 4097, "none"), (20, 6000, "none"), (21, 6000, "tile 16x16"), (24, 8192, "tile 16x16"),
    (24, 8193, "none"), (36, 5456, "tile 16x16"), (36, 5457, "none"), (37, 5457, "tile 16x16"), (7, 100000, "none")])
def test_forms_of_few_columns(lx, ly, form):
    assert lattice(lx, ly, precision="fp32").two_step_form() == form
    assert lattice(lx, ly, precision="fp32_f32sums").two_step_form() == "tile 16x16"
    assert lattice(lx, ly, precision="fp64").two_step_form() == "tile 16x16"
