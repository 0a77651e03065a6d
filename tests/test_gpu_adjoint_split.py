"""The adjoint step's two launch forms agree: small lattices give every row
segment a wavefront of its own, larger ones walk eight segments per block.

A lattice made of k copies of a small one along z is periodic in the copy, so its
adjoint is the small one's in every copy and its rate gradient k times the small
one's.  k is chosen so that the copies run in the other form.  Sizes: one and two
64-lane columns, a last column of one lane, a full 256-node block, rows of three
nodes, fewer row segments than the eight of a block.

Tolerances: FP64, 1e-13 of the largest entry (lambda, dL/dF: the same arithmetic
in another kernel, a few roundings) and 1e-12 of the sum of the magnitudes for the
summed gradients (10^5 terms added in another order: n eps / 2 at worst 1e-11, its
square root 2e-14 as a rule).  FP32, 2e-6 of the largest entry (16 roundings of
2^-24), and for the summed gradients 8 roundings of 2^-24 per thread's sum, 5e-7.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_setup

pytestmark = pytest.mark.gpu

F64, F32 = 0, 1


def _adjoint(q, prec, shape, copies, solid, field, f, lam, rates):
    shape = (shape[0] * copies,) + shape[1:]
    rep = (1, copies, 1, 1)
    F = np.tile(field, rep) if field.ndim == 4 else field
    sim = gpu_setup(q, shape, prec, rates, F, None if solid is None else np.tile(solid, rep[1:]))
    x = sim.import_populations(f.repeat(rep))
    lam, out = lam.repeat(rep).contiguous(), sim.real_populations()
    dF = torch.zeros((3,) + shape if field.ndim == 4 else 3, dtype=torch.float64, device="cuda")
    dw = torch.zeros(q - 4, dtype=torch.float64, device="cuda")
    out.zero_()
    sim.adjoint_step(x, lam, out, dF, dw)
    return out.double(), dF, dw


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec", [F32, F64], ids=["f32", "f64"])
@pytest.mark.parametrize("q", [27, 15])
def test_both_forms_agree(q, prec, walls):
    blocks = 4096 if q == 15 and prec == F32 else 1024
    for i, shape in enumerate([(1, 1, 64), (2, 3, 65), (3, 5, 130), (2, 6, 256), (5, 4, 3), (3, 1, 300)]):
        print(f"case q{q} prec{prec} {shape} walls={walls}", flush=True)
        nz, ny, nx = shape
        rng = np.random.default_rng(i)
        solid = rng.random(shape) < 0.1 if walls else None
        F = 1e-3 * rng.standard_normal((3,) + shape) if i % 2 else np.array([2e-3, -1e-3, 5e-4])
        rates = list(rng.uniform(0.7, 1.9, q - 4))
        real = torch.float64 if prec == F64 else torch.float32
        w = torch.tensor([8 / 27] + [2 / 27] * 6 + [1 / 54] * 12 + [1 / 216] * 8 if q == 27
                         else [2 / 9] + [1 / 9] * 6 + [1 / 72] * 8)
        f = (w[:, None, None, None] * torch.from_numpy(1 + 0.1 * rng.standard_normal((q,) + shape))).to("cuda", real)
        lam = torch.from_numpy(rng.standard_normal((q,) + shape)).to("cuda", real)
        segments = -(-nx // 256) * -(-min(nx, 256) // 64) * ny * nz       # 64-lane columns
        k = 8 * (blocks + 16) // segments + 1
        few = _adjoint(q, prec, shape, 1, solid, F, f, lam, rates)
        many = _adjoint(q, prec, shape, k, solid, F, f, lam, rates)
        entry, total = (1e-13, 1e-12) if prec == F64 else (2e-6, 5e-7)
        for a, b, fields in zip(few[:2], many[:2], (True, i % 2)):
            if fields:
                b = b.reshape(b.shape[0], k, *shape)
                assert float((b - a[:, None]).abs().max()) <= entry * float(a.abs().max())
            else:
                assert float((b / k - a).abs().max()) <= total * float(lam.double().abs().sum())
        assert float((many[2] / k - few[2]).abs().max()) <= total * float(lam.double().abs().sum())
