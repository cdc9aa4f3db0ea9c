"""The rule that cuts FP64 outputs into tiles (CPU): every element belongs to
one tile, and each kind of tile is taken where its rule says."""
import numpy as np
import pytest

from paper_2309_16724_amd import binding as B
from paper_2309_16724_amd.synth.problem import random_problem

SIZES = (1, 4, 15, 16, 17, 33, 47, 48, 49, 63, 64, 65, 95, 96, 97, 127, 128, 129, 175, 176, 191, 192, 193, 257, 520)
SHAPE = {1: (16, 64), 2: (32, 32), 4: (64, 16), 8: (64, 64), 32: (128, 128)}


@pytest.mark.parametrize("m", SIZES)
def test_tiles_cover_the_output_once(m):
    for n in SIZES:
        seen = np.zeros((m, n), dtype=np.int8)
        for i0, j0, kind in B.debug_f64_cells(m, n):
            rows, cols = SHAPE[int(kind)]
            seen[i0:i0 + rows, j0:j0 + cols] += 1
        assert seen.min() == 1 and seen.max() == 1, (m, n)


@pytest.mark.parametrize("m,n,kinds", [
    (48, 48, {8}), (47, 48, {2}), (48, 47, {2}), (47, 300, {2}), (63, 300, {8}),
    (64, 95, {8}), (64, 96, {32}), (96, 64, {32}), (63, 96, {8}),
    (16, 300, {1}), (300, 16, {4}), (17, 17, {2}),
    (128, 128, {32}), (192, 128, {32}), (191, 128, {8, 32}), (175, 128, {2, 32}), (130, 300, {1, 2, 32}),
])
def test_tile_kinds(m, n, kinds):
    assert set(B.debug_f64_cells(m, n)[:, 2]) == kinds


def test_plans_of_the_gpu_tests_have_every_kind():
    """The shapes that test_gpu_tile_edges.py compares with the oracle reach
    all five kinds (the 128 x 128 one in the first stage; the second stage's are
    in test_gpu_wg_tiles.py)."""
    seen = set()
    for D, Dr in ((300, 300), (340, 700), (620, 150), (160, 640)):
        prob = random_problem(6, 6, 0, 5, D=D, D_right=Dr, cap=False)
        first = set(B.debug_plan_tiles(prob, 1)[:, 6])
        assert 32 in first, (D, Dr, first)
        seen |= first | set(B.debug_plan_tiles(prob, 2)[:, 6])
    assert seen == {1, 2, 4, 8, 32}


def test_small_chunks_and_long_parts_take_small_tiles():
    """Few outputs at a time leave no room for large tiles: a plan in one chunk
    has 128 x 128 tiles in both stages, in chunks of 8 MiB none (64 x 64 ones in a
    few chunks), and with parts of 16384 along K none in the second stage."""
    prob = random_problem(6, 6, 0, 1, D=600, cap=False)

    def kinds(stage, **kw):
        return set(B.debug_plan_tiles(prob, stage, **kw)[:, 6])

    assert 32 in kinds(1) and 32 in kinds(2)
    assert 32 not in kinds(1, workspace_bytes=8 << 20) | kinds(2, workspace_bytes=8 << 20)
    assert 32 in kinds(1, kpart=16384) and 32 not in kinds(2, kpart=16384)
