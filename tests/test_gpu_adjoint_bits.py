"""The adjoint step's launch forms give the same bits.

  * Rows of 64 nodes and the same rows twice over (128 nodes, periodic): as many row
    segments in the same blocks, but the second lattice runs in the other form, and each of
    its sums is twice the first's, exactly: dL/domega and a uniform force's dL/dF are
    compared bit for bit, lambda too.
  * A lattice and its copies along z, in the other form: lambda and dL/dF of a force
    field, node by node.  Among them rows of 300, 320 and 513 nodes whose segments are
    equal (192 + 128 nodes and less, instead of 256 and a remainder) and some whose are not.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_setup
from plan_helpers import adjoint_launch

pytestmark = pytest.mark.gpu

F64, F32, F16DEV, BF16DEV = 0, 1, 2, 3
KINDS = pytest.mark.parametrize("q,prec,per_mass", [(27, F32, False), (27, F32, True), (27, F64, False), (27, F64, True),
                                                    (15, F32, True), (15, F32, False), (15, F64, True), (27, F16DEV, False),
                                                    (15, BF16DEV, True)])
WALLS = pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])


def _inputs(q, prec, shape, walls, seed):
    rng = np.random.default_rng(seed)
    real = torch.float64 if prec == F64 else torch.float32
    w = torch.tensor([8 / 27] + [2 / 27] * 6 + [1 / 54] * 12 + [1 / 216] * 8 if q == 27
                     else [2 / 9] + [1 / 9] * 6 + [1 / 72] * 8)
    f = (w[:, None, None, None] * torch.from_numpy(1 + 0.1 * rng.standard_normal((q,) + shape))).to("cuda", real)
    lam = torch.from_numpy(rng.standard_normal((q,) + shape)).to("cuda", real)
    solid = torch.from_numpy(rng.random(shape) < 0.1).to("cuda", torch.uint8) if walls else None
    field = torch.from_numpy(1e-2 * rng.standard_normal((3,) + shape)).to("cuda", real)
    return f, lam, solid, field, list(rng.uniform(0.7, 1.9, q - 4))


def _adjoint(q, prec, per_mass, f, lam, solid, force, rates, scale=1.0):
    shape = tuple(f.shape[1:])
    sim = gpu_setup(q, shape, prec, rates, per_mass=per_mass)
    if solid is not None:
        sim.set_mask(solid)
    sim.set_force(force)
    sim.set_force_scale(scale)
    field = isinstance(force, torch.Tensor)
    dF = torch.zeros((3,) + shape if field else 3, dtype=torch.float64, device="cuda")
    dw = torch.zeros(q - 4, dtype=torch.float64, device="cuda")
    out = sim.real_populations().zero_()
    sim.adjoint_step(sim.import_populations(f), lam, out, dF, dw)
    return out, dF, dw


@WALLS
@KINDS
def test_sums_of_both_forms(q, prec, per_mass, walls):
    rows = (144, 128) if q == 15 and prec != F64 else (72, 64)
    one, two = adjoint_launch(q, prec, rows + (64,)), adjoint_launch(q, prec, rows + (128,))
    assert one.split and not two.split and one.blocks == two.blocks
    print(f"case q{q} prec{prec} {rows} walls={walls}", flush=True)
    f, lam, solid, _, rates = _inputs(q, prec, rows + (64,), walls, 1)
    force = [2e-3, -1e-3, 5e-4]
    a = _adjoint(q, prec, per_mass, f, lam, solid, force, rates, scale=0.75)
    b = _adjoint(q, prec, per_mass, f.repeat(1, 1, 1, 2).contiguous(), lam.repeat(1, 1, 1, 2).contiguous(),
                 None if solid is None else solid.repeat(1, 1, 2).contiguous(), force, rates, scale=0.75)
    assert torch.equal(b[0], a[0].repeat(1, 1, 1, 2))
    assert torch.equal(b[1], 2 * a[1])
    assert torch.equal(b[2], 2 * a[2])


@WALLS
@KINDS
def test_nodes_of_both_forms(q, prec, per_mass, walls):
    for i, (shape, equal) in enumerate([((1, 1, 64), False), ((2, 3, 65), False), ((3, 5, 130), False), ((2, 6, 256), False),
                                        ((5, 4, 3), False), ((3, 1, 300), False), ((8, 6, 300), True), ((8, 6, 320), True),
                                        ((8, 8, 513), True)]):
        few = adjoint_launch(q, prec, shape)
        copies = next(k for k in range(2, 100000)
                      if not (m := adjoint_launch(q, prec, (k * shape[0],) + shape[1:])).split
                      and (m.segment < 256) == (equal or shape[2] < 193))
        assert few.split and (few.segment < 256) == (equal or shape[2] < 193), (shape, few)
        print(f"case q{q} prec{prec} {shape} x {copies} walls={walls}", flush=True)
        f, lam, solid, field, rates = _inputs(q, prec, shape, walls, i)
        a = _adjoint(q, prec, per_mass, f, lam, solid, field, rates, scale=0.75)
        rep = (1, copies, 1, 1)
        b = _adjoint(q, prec, per_mass, f.repeat(rep), lam.repeat(rep).contiguous(),
                     None if solid is None else solid.repeat(rep[1:]).contiguous(), field.repeat(rep).contiguous(), rates,
                     scale=0.75)
        for x, y in zip(a[:2], b[:2]):
            assert torch.equal(y, x.repeat(rep)), shape
