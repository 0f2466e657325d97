"""Structured layout at the edges of the tile sort: numbers of distinct cells
at and across one and two six-bit passes and the small table's limit, with and
without unplaced voxels, ordered and shuffled, and a ragged last tile.  The
layout is a permutation: compared exactly with the oracle's stable sorts."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import banner
from tests.test_gpu_layout import _check

pytestmark = pytest.mark.gpu
TILE = 4096


@pytest.mark.parametrize("distinct", [1, 2, 62, 63, 64, 639, 640, 641, 4095])
@pytest.mark.parametrize("none", [False, True])
def test_tile_sort_edges(distinct, none):
    rng = np.random.default_rng(distinct + 7 * none)
    shape = (1, 3, 2817)  # two tiles and 259 voxels of a third
    n = int(np.prod(shape))
    S = 5000
    cell = np.empty(n, dtype=np.uint32)
    for tile, v in enumerate(range(0, n, TILE)):
        k = min(TILE, n - v)
        ids = rng.choice(S, size=min(distinct, k), replace=False).astype(np.uint32)
        c = np.sort(np.concatenate([np.arange(len(ids)), rng.integers(0, len(ids), size=k - len(ids))]))
        if tile:
            c = rng.permutation(c)
        cell[v:v + k] = ids[c]
    if none:
        cell[rng.random(n) < 0.1] = oracle.NONE_ID
        cell[5] = S + 3  # an id past the last cell is not placed either
    site_comp = rng.integers(0, 9, size=S).astype(np.uint32)
    comp_band = np.sort(rng.integers(0, 3, size=9)).astype(np.uint8)
    banner(f"tile sort: {distinct} cells a tile, none={none}")
    _check(cell.reshape(shape), site_comp, comp_band, 9, 3, shape)
