"""Rows of more than 256 nodes: a plain step and an in-place step cut them into equal
blocks of one to four wavefronts, a step with totals into as few as blocks of four
give, and the adjoint likewise.

The populations of the plain step, of the step with totals and of the in-place
scheme agree bit for bit (the other tests compare them with the oracle at up to
300 nodes).  Sizes: 5 to 13 wavefronts per row, of which 5, 7, 11 and 13 are cut one by
one, 6 and 9 by threes, 10 by twos; a last wavefront of one node and a full one.  The
adjoint's two launch forms agree within test_gpu_adjoint_split's tolerances.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_setup
from test_gpu_adjoint_split import _adjoint

pytestmark = pytest.mark.gpu

F64, F32, F16DEV, BF16DEV = 0, 1, 2, 3
WIDTHS = [257, 300, 320, 321, 384, 400, 448, 513, 640, 650, 770]


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec", [F64, F32, F16DEV, BF16DEV], ids=["f64", "f32", "f16dev", "bf16dev"])
@pytest.mark.parametrize("q", [27, 15])
def test_step_forms_agree_bit_for_bit(q, prec, walls):
    for i, nx in enumerate(WIDTHS):
        shape = (3, 2, nx) if i % 2 else (2, 5, nx)
        rng = np.random.default_rng(i)
        solid = rng.random(shape) < 0.08 if walls else None
        F = 1e-4 * rng.standard_normal((3,) + shape) if i % 3 else np.array([2e-4, -1e-4, 5e-5])
        sim = gpu_setup(q, shape, prec, list(rng.uniform(0.7, 1.9, q - 4)), F, solid)
        rho = torch.from_numpy(1 + 0.01 * rng.standard_normal(shape)).cuda()
        u = torch.from_numpy(0.05 * rng.uniform(-1, 1, (3,) + shape)).cuda()
        a = sim.init_equilibrium(rho, u)[0]
        buf = sim.init_equilibrium_inplace(rho, u)
        b, totals = a.clone(), torch.zeros(4, dtype=torch.float64, device="cuda")
        for _ in range(2):
            a2, b2 = torch.zeros_like(a), torch.zeros_like(b)
            sim.step(a, a2)
            sim.step(b, b2, totals=totals)
            a, b = a2, b2
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (shape, prec)
        sim.run_inplace(buf, 2)
        fluid = slice(None) if solid is None else torch.from_numpy(~solid).cuda()
        assert torch.equal(sim.gather(a)[:, fluid], sim.export_populations(buf)[:, fluid]), (shape, prec)


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec", [F32, F64], ids=["f32", "f64"])
@pytest.mark.parametrize("q", [27, 15])
def test_adjoint_forms_agree(q, prec, walls):
    real, entry, total = (torch.float64, 1e-13, 1e-12) if prec == F64 else (torch.float32, 2e-6, 5e-7)
    for i, shape in enumerate([(3, 1, 300), (2, 2, 320), (1, 2, 513)]):
        rng = np.random.default_rng(i)
        solid = rng.random(shape) < 0.1 if walls else None
        F, rates = 1e-3 * rng.standard_normal((3,) + shape), list(rng.uniform(0.7, 1.9, q - 4))
        w = torch.tensor([8 / 27] + [2 / 27] * 6 + [1 / 54] * 12 + [1 / 216] * 8 if q == 27
                         else [2 / 9] + [1 / 9] * 6 + [1 / 72] * 8)
        f = (w[:, None, None, None] * torch.from_numpy(1 + 0.1 * rng.standard_normal((q,) + shape))).to("cuda", real)
        lam = torch.from_numpy(rng.standard_normal((q,) + shape)).to("cuda", real)
        # eight segments a block of three columns of 64 lanes, or more: beyond the split form's blocks
        segments = -(-shape[2] // 256) * shape[0] * shape[1]
        k = 8 * ((4096 if q == 15 and prec == F32 else 1024) // 3 + 16) // segments + 1
        few = _adjoint(q, prec, shape, 1, solid, F, f, lam, rates)
        many = _adjoint(q, prec, shape, k, solid, F, f, lam, rates)
        for a, b in zip(few[:2], many[:2]):
            b = b.reshape(b.shape[0], k, *shape)
            assert float((b - a[:, None]).abs().max()) <= entry * float(a.abs().max())
        assert float((many[2] / k - few[2]).abs().max()) <= total * float(lam.double().abs().sum())
