"""cmlbm_run's two steps in one pass: the populations of both buffers bit for bit
those of as many cmlbm_step calls (which the other tests compare with the
oracle), on lattices just large enough to be run that way.

Sizes: a tile is 64 nodes by 8 (or 4) rows and walks along z; a last block of fewer
than 64 nodes is packed over the threads or, where nearly full, is not; rows left
over in y; one plane, one row and two rows (the halo is the tile itself); rows of
a few nodes.  With walls, a solid plane at each end of an axis and solid nodes at
random, so that every direction bounces at tile edges and inside.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_setup

pytestmark = pytest.mark.gpu

F64, F32 = 0, 1
SHAPES = [                       # nz, ny, nx
    (64, 64, 64), (1, 515, 512), (515, 1, 512), (530, 2, 256), (33, 66, 128),
    (68, 60, 65), (67, 61, 66), (45, 47, 127), (40, 67, 100), (16, 130, 130), (61, 69, 63), (100, 90, 33),
    (64, 64, 3), (90, 50, 7), (128, 128, 1),
]


def _state(sim, shape, seed, nan):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rho = 1 + 0.01 * torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)
    u = 0.05 * (torch.rand((3,) + shape, generator=gen, device="cuda", dtype=torch.float64) - 0.5)
    f, _ = sim.init_equilibrium(rho, u)
    if nan:
        f.view(-1)[f.numel() // 2] = float("nan")
    return f


def _run_both(q, prec, shape, walls, field, steps, nan=False):
    rng = np.random.default_rng(5)
    solid = None
    if walls:
        solid = rng.random(shape) < 0.02
        solid[0] = solid[-1] = True
    F = 1e-4 * rng.standard_normal((3,) + shape) if field else np.array([2e-4, -1e-4, 5e-5])
    sim = gpu_setup(q, shape, prec, list(rng.uniform(0.7, 1.9, q - 4)), F, solid)
    a = _state(sim, shape, 11, nan)
    b = torch.zeros_like(a)
    want = [a.clone(), b.clone()]
    for n in range(steps):
        sim.step(want[n & 1], want[(n + 1) & 1])
    last = sim.run(a, b, steps)
    assert last is (b if steps & 1 else a)
    return (a, b), want


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec", [F32, F64], ids=["f32", "f64"])
@pytest.mark.parametrize("q", [27, 15])
def test_run_is_its_single_steps_bit_for_bit(q, prec, walls):
    for i, shape in enumerate(SHAPES):
        if prec == F32 and q == 15 and walls:
            shape = (2 * shape[0],) + shape[1:]            # (that one starts at 2^19 nodes)
        print(f"case q{q} prec{prec} {shape} walls={walls}", flush=True)
        got, want = _run_both(q, prec, shape, walls, field=i % 2 == 0, steps=5 + i % 4)
        for g, w in zip(got, want):
            assert torch.equal(g, w), shape


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
def test_a_nan_spreads_as_in_single_steps(walls):
    print(f"case nan walls={walls}", flush=True)
    got, want = _run_both(27, F32, (40, 67, 100), walls, field=True, steps=6, nan=True)
    for g, w in zip(got, want):
        assert int(torch.isnan(w).sum()) > 27
        assert torch.equal(torch.isnan(g), torch.isnan(w))
        assert torch.equal(torch.nan_to_num(g), torch.nan_to_num(w))
