"""Where cmlbm_run takes two steps in one pass over the populations (host rule).

A block of that pass walks a tile of 64 nodes by 8 (or 4) rows along z and
collides its halo too, so that lattices of a few rows or planes, or of few tiles
and many planes, take longer than in single steps: the rule has to leave those
alone, and to take the lattices that fill the tiles.
"""
import timeit

import pytest

from plan_helpers import lib, step2_plan

F64, F32, F16DEV, BF16DEV = 0, 1, 2, 3

# (nx, ny, nz) that took 1.2 to 9 times as long as single steps
FLAT = [(512, 515, 1), (2048, 2048, 1), (8192, 512, 1), (100, 2700, 1), (9, 30000, 1),
        (512, 1, 515), (2048, 1, 2048), (64, 1, 4096), (100, 1, 2700), (9, 1, 30000),
        (4, 4, 16384), (8, 8, 8192), (8, 8, 65535), (9, 4, 30000)]
# ... and that gain in every kind
ROOMY = [(256, 128, 16), (256, 256, 8), (512, 512, 4), (256, 8, 256), (512, 4, 512), (40, 200, 200), (24, 200, 200),
         (9, 400, 400), (12, 300, 300), (128, 128, 128), (201, 131, 67), (384, 300, 300), (512, 512, 512)]
# (nz, ny, nx) that the GPU tests run, in every kind and in those that gain
REACHED = [(500, 601, 2), (300, 258, 7), (512, 4, 512), (520, 4, 1000), (260, 63, 63), (67, 66, 128), (80, 67, 100),
           (530, 8, 257), (200, 191, 65), (90, 130, 130), (200, 91, 33)]
REACHED_BY_SOME = [(1025, 520, 1), (700, 701, 1), (170, 150, 10), (140, 130, 11), (130, 127, 15), (600, 3, 1100),
                   (600, 2, 2000), (3, 700, 512), (2000, 17, 19), (64, 64, 64)]


@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("prec", [F64, F32])
@pytest.mark.parametrize("q", [27, 15])
def test_thin_lattices_keep_single_steps(q, prec, walls):
    for nx, ny, nz in FLAT:
        assert not step2_plan(q, prec, (nz, ny, nx), walls).pays, (nx, ny, nz)


@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("prec", [F64, F32])
@pytest.mark.parametrize("q", [27, 15])
def test_lattices_that_fill_the_tiles_take_two_steps(q, prec, walls):
    for nx, ny, nz in ROOMY:
        assert step2_plan(q, prec, (nz, ny, nx), walls).pays, (nx, ny, nz)


@pytest.mark.parametrize("q", [27, 15])
def test_limits(q):
    for prec in (F16DEV, BF16DEV):
        assert not step2_plan(q, prec, (512, 512, 512), 0).pays
    for prec in (F64, F32):
        assert not step2_plan(q, prec, (56, 56, 56), 0).pays
        # offsets inside a plane of population rows have 32 bits
        ny = (2**32 // (8 if prec == F64 else 4) // q - 1) // 4096
        assert step2_plan(q, prec, (8, ny, 4096), 0).pays
        assert not step2_plan(q, prec, (8, ny + 1, 4096), 0).pays


def _planes_per_block(tiles, nz):
    """Every plane count tried: rounds of 256 blocks, each its planes and three more."""
    return min(range(nz, 0, -1), key=lambda z: -(-tiles * -(-nz // z) // 256) * (z + 3))


def test_planes_per_block_are_the_best_of_all():
    for tiles in [*range(1, 30), 64, 100, 127, 128, 129, 200, 255, 256, 257, 300, 511, 512, 1000, 4096, 70000]:
        for nz in [*range(1, 20), 64, 67, 100, 255, 256, 257, 600, 1021]:
            assert lib().hp_run_length(tiles, nz) == _planes_per_block(tiles, nz), (tiles, nz)


def test_planes_per_block_take_no_time_on_tall_lattices():
    # cmlbm_run asks once per call, where a step takes 5 us at least
    for tiles in (1, 2, 7, 100, 129, 200, 255, 256, 300, 1000):
        best = min(timeit.repeat(lambda: lib().hp_run_length(tiles, 65535), number=20, repeat=5)) / 20
        assert best < 20e-6, (tiles, best)


def test_the_lattices_of_the_gpu_tests_are_reached():
    kinds = [(q, prec, walls) for q in (27, 15) for prec in (F64, F32) for walls in (0, 1)]
    for shape in REACHED:
        assert all(step2_plan(q, prec, shape, walls).pays for q, prec, walls in kinds), shape
    for shape in REACHED_BY_SOME:
        assert any(step2_plan(q, prec, shape, walls).pays for q, prec, walls in kinds), shape
    for q, prec, walls in kinds:
        some = [s for s in REACHED_BY_SOME if step2_plan(q, prec, s, walls).pays]
        assert len(some) >= 2, (q, prec, walls)
        tiles = [step2_plan(q, prec, s, walls) for s in REACHED + some]
        assert any(t.main and t.tail for t in tiles) and any(not t.main for t in tiles) and any(not t.tail for t in tiles)
