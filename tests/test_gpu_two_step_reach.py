"""cmlbm_run's two steps in one pass on lattices that its rule sends there (asked of
the rule itself): the populations of both buffers bit for bit those of as many
cmlbm_step calls.

Sizes: rows of one, two and seven nodes, whose halo columns are the tile's own; a
short last block packed beside full ones and one that is not; rows left over in y;
fewer rows than a tile's; a few planes; under 2^18 nodes, where rows of 10 to 15 nodes
are sent there; and planes of 2 to 4 GiB of populations, whose offsets need the
32nd bit.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_setup
from plan_helpers import step2_plan
from test_step2_plan import REACHED, REACHED_BY_SOME

pytestmark = pytest.mark.gpu

F64, F32 = 0, 1


def _sim(q, prec, shape, walls, field):
    rng = np.random.default_rng(5)
    gen = torch.Generator(device="cuda").manual_seed(11)

    def rand(*size):
        return torch.rand(size, generator=gen, device="cuda", dtype=torch.float64)

    sim = gpu_setup(q, shape, prec, list(rng.uniform(0.7, 1.9, q - 4)))
    if walls:
        solid = rand(*shape) < 0.02
        solid[0] = True
        solid[:, :, -1] |= rand(*shape[:2]) < 0.5
        sim.set_mask(solid.to(torch.uint8))
    sim.set_force(1e-4 * (rand(3, *shape) - 0.5) if field else [2e-4, -1e-4, 5e-5])
    f, _ = sim.init_equilibrium(1 + 0.01 * rand(*shape), 0.05 * (rand(3, *shape) - 0.5))
    return sim, f


def _check(q, prec, shape, walls, field, steps):
    print(f"case q{q} prec{prec} {shape} walls={walls} field={field}", flush=True)
    sim, a = _sim(q, prec, shape, walls, field)
    b = torch.zeros_like(a)
    want = [a.clone(), b.clone()]
    for n in range(steps):
        sim.step(want[n & 1], want[(n + 1) & 1])
    assert sim.run(a, b, steps) is (b if steps & 1 else a)
    assert torch.equal(a, want[0]) and torch.equal(b, want[1]), shape


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec", [F32, F64], ids=["f32", "f64"])
@pytest.mark.parametrize("q", [27, 15])
def test_run_is_its_single_steps_bit_for_bit(q, prec, walls):
    for shape in REACHED:
        assert step2_plan(q, prec, shape, walls).pays, shape
    reached = REACHED + [s for s in REACHED_BY_SOME if step2_plan(q, prec, s, walls).pays]
    for i, shape in enumerate(reached):
        _check(q, prec, shape, walls, field=i % 2 == 0, steps=5 + i % 4)


@pytest.mark.parametrize("q,prec,shape,walls", [(27, F64, (4, 3000, 4100), False), (27, F32, (4, 5003, 6000), True)],
                         ids=["f64", "f32-walls"])
def test_planes_of_more_than_two_gib(q, prec, shape, walls):
    assert 2**31 < shape[1] * shape[2] * q * (8 if prec == F64 else 4) < 2**32
    assert step2_plan(q, prec, shape, walls).pays
    _check(q, prec, shape, walls, field=prec == F64, steps=5)
    torch.cuda.empty_cache()
