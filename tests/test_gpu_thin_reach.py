"""Where the step begins to take its nodes in a row (asked of the rule itself), and one
row before: the populations bit for bit those of the step with totals, which keeps a
wavefront per row.
"""
import pytest
import torch

from plan_helpers import thin_pays
from test_gpu_thin_step import _setup

pytestmark = pytest.mark.gpu

# rows at which each kind begins, for 13 nodes a row: (q, bytes, walls)
BEGIN = {(27, 8, False): 4096, (15, 8, False): 8192, (27, 4, False): 10240, (15, 4, False): 16384,
         (27, 2, False): 8192, (15, 2, False): 4096}


@pytest.mark.parametrize("walls", [False, True], ids=["periodic", "walls"])
@pytest.mark.parametrize("prec", [0, 1, 2, 3], ids=["f64", "f32", "f16dev", "bf16dev"])
@pytest.mark.parametrize("q", [27, 15])
def test_thin_step_where_it_begins(q, prec, walls):
    rows = 4096 if walls else BEGIN[q, (8, 4, 2, 2)[prec], False]
    for shape, thin in [((rows // 64, 64, 13), True), ((1, rows - 1, 13), False)]:
        assert thin_pays(q, prec, shape, walls) == thin
        sim, f = _setup(q, prec, shape, walls, field=True)
        totals = torch.zeros(4, dtype=torch.float64, device="cuda")
        a, b = torch.zeros_like(f), torch.zeros_like(f)
        sim.step(f, a)
        sim.step(f, b, totals=totals)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (shape, prec)
