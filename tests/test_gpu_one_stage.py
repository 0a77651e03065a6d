"""Sums of block partials, in one launch up to a number of rows and in two beyond: the
totals of a step (3584 rows) and the rate and force gradients of an adjoint step
(6144), at the last row count of the one and the first of the other (the next multiple of its
copies for the adjoint).

The references are sums of the library's other outputs in FP64 by torch: the totals of
the gathered populations, and the gradients of a lattice of 8 planes times its copies.
Tolerance: the terms are the same, added in another order; n eps / 2 of the sum of
their magnitudes bounds the difference of two orders, n the most that one chain adds (below
100 here), so 100 eps = 2e-14 of that sum.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import gpu_setup

pytestmark = pytest.mark.gpu

F64 = 0


@pytest.mark.parametrize("rows", [3584, 3585])
@pytest.mark.parametrize("q", [27, 15])
def test_step_totals(q, rows):
    shape = (rows, 1, 32)
    rng = np.random.default_rng(2)
    sim = gpu_setup(q, shape, F64, list(rng.uniform(0.7, 1.9, q - 4)))
    sim.set_force(torch.from_numpy(1e-3 * rng.standard_normal((3,) + shape)))
    f = sim.init_equilibrium(torch.from_numpy(1 + 0.1 * rng.standard_normal(shape)).cuda(),
                             torch.from_numpy(0.05 * rng.standard_normal((3,) + shape)).cuda())[0]
    totals = torch.full((4,), float("nan"), dtype=torch.float64, device="cuda")
    sim.step(f, torch.zeros_like(f), totals=totals)
    rho, u = sim.macroscopic(f)
    terms = torch.stack([rho, *(rho * u)]).double().reshape(4, -1)
    # (rho u is j of the FP64 populations after two roundings of a term)
    assert ((totals - terms.sum(1)).abs() <= 2e-14 * terms.abs().sum(1) + 4 * 2.0**-53 * terms.abs().sum(1)).all()


@pytest.mark.parametrize("blocks", [6144, 6208])
@pytest.mark.parametrize("q", [27, 15])
def test_adjoint_gradients(q, blocks):
    def gradients(planes, f, lam):
        shape = (planes, 64, 3)
        sim = gpu_setup(q, shape, F64, rates)
        sim.set_force([2e-3, -1e-3, 5e-4])
        dF = torch.zeros(3, dtype=torch.float64, device="cuda")
        dw = torch.zeros(q - 4, dtype=torch.float64, device="cuda")
        copies = (1, planes // 8, 1, 1)
        sim.adjoint_step(sim.import_populations(f.repeat(copies)), lam.repeat(copies).contiguous(), sim.real_populations(),
                         dF, dw)
        return torch.cat([dF, dw])

    rng = np.random.default_rng(3)
    rates = list(rng.uniform(0.7, 1.9, q - 4))
    f = torch.from_numpy(0.05 + 0.005 * rng.standard_normal((q, 8, 64, 3))).cuda()
    lam = torch.from_numpy(rng.standard_normal((q, 8, 64, 3))).cuda()
    planes = blocks * 8 // 64
    one, many = gradients(8, f, lam), gradients(planes, f, lam)
    # |dL/domega_b| and |dL/dF| of a node are below the sum of its |lambda|
    assert float((many * (8 / planes) - one).abs().max()) <= 2e-14 * float(lam.abs().sum())
