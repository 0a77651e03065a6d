"""Which steps take their nodes in a row, whatever rows they are in (host rule)."""
import pytest

from plan_helpers import thin_pays

F64, F32, F16DEV, BF16DEV = 0, 1, 2, 3
KINDS = [(q, prec, walls) for q in (27, 15) for prec in range(4) for walls in (0, 1)]


@pytest.mark.parametrize("q,prec,shape", [(27, F32, (76, 77, 15)), (27, F32, (70, 71, 13)), (27, F32, (64, 64, 14)),
                                          (15, F32, (97, 98, 15)), (15, F32, (84, 85, 13)), (15, F32, (104, 105, 13)),
                                          (15, F64, (76, 77, 15)), (27, F16DEV, (76, 77, 15)), (27, BF16DEV, (70, 71, 13))])
def test_rows_that_were_faster_keep_their_wavefronts(q, prec, shape):
    """These took 1.07 to 1.3 times as long with their nodes in a row."""
    assert not thin_pays(q, prec, shape, 0)


def test_where_taking_nodes_in_a_row_wins():
    for q, prec, walls in KINDS:
        assert thin_pays(q, prec, (45, 45, 3), walls) and thin_pays(q, prec, (40, 40, 8), walls)      # 0.5-0.98
        assert thin_pays(q, prec, (140, 141, 13), walls)                                              # 0.52-0.92
        assert not thin_pays(q, prec, (45, 3, 3), walls) and not thin_pays(q, prec, (40, 40, 9), walls)
        assert not thin_pays(q, prec, (200, 200, 33), walls)
        assert thin_pays(q, prec, (128, 128, 32), walls) == (prec >= F16DEV)
