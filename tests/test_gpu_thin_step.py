"""The step that takes nodes in a row, whatever rows of the lattice they are in (few
nodes in x): the populations bit for bit those of a step with totals, which keeps
a wavefront per row and which the other tests compare with the oracle.

Sizes: one node per row up to the widest of each rule, row counts at which the rule
begins, last wavefronts of one node and of 63, one plane; and a run of steps on a thin
lattice large enough for two steps per pass.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_setup

pytestmark = pytest.mark.gpu

F64, F32, F16DEV, BF16DEV = 0, 1, 2, 3
SHAPES = [(32, 48, 1), (45, 35, 3), (41, 43, 5), (1, 2049, 7), (40, 40, 8), (64, 64, 9), (67, 67, 13), (66, 65, 16)]
NARROW = [(128, 128, 17), (131, 127, 32)]


def _setup(q, prec, shape, walls, field):
    rng = np.random.default_rng(9)
    solid = None
    if walls:
        solid = rng.random(shape) < 0.05
        solid[:, 0] = solid[:, -1] = True
    F = 1e-4 * rng.standard_normal((3,) + shape) if field else np.array([2e-4, -1e-4, 5e-5])
    sim = gpu_setup(q, shape, prec, list(rng.uniform(0.7, 1.9, q - 4)), F, solid)
    gen = torch.Generator(device="cuda").manual_seed(3)
    rho = 1 + 0.01 * torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)
    u = 0.05 * (torch.rand((3,) + shape, generator=gen, device="cuda", dtype=torch.float64) - 0.5)
    return sim, sim.init_equilibrium(rho, u)[0]


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec", [F64, F32, F16DEV, BF16DEV], ids=["f64", "f32", "f16dev", "bf16dev"])
@pytest.mark.parametrize("q", [27, 15])
def test_thin_step_is_the_row_step_bit_for_bit(q, prec, walls):
    for i, shape in enumerate(SHAPES + (NARROW if prec >= F16DEV else [])):
        sim, f = _setup(q, prec, shape, walls, field=bool(i & 1))
        totals = torch.zeros(4, dtype=torch.float64, device="cuda")
        a, b = f, f.clone()
        for _ in range(2):
            a2, b2 = torch.zeros_like(a), torch.zeros_like(b)
            sim.step(a, a2)
            sim.step(b, b2, totals=totals)
            a, b = a2, b2
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (shape, prec)


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("q", [27, 15])
def test_thin_run_is_its_single_steps_bit_for_bit(q, walls):
    for prec in (F64, F32):
        sim, f = _setup(q, prec, (420, 419, 3), walls, field=False)
        want, b = [f.clone(), torch.zeros_like(f)], torch.zeros_like(f)
        for n in range(6):
            sim.step(want[n & 1], want[(n + 1) & 1])
        assert sim.run(f, b, 6) is f
        assert torch.equal(f.view(torch.uint8), want[0].view(torch.uint8))
        assert torch.equal(b.view(torch.uint8), want[1].view(torch.uint8))
