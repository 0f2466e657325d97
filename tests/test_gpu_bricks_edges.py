"""Brick relaxation at the edges of its bricks: volumes one voxel short of, at
and past whole 16^3 bricks on each axis, thin ones, bands that change at every
voxel and bands of one value, both key widths, one pass and an update loop,
bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 16, 17), (15, 16, 17), (16, 16, 16), (17, 33, 1), (31, 15, 48),
                                   (33, 17, 34), (17, 20, 2100)])
@pytest.mark.parametrize("n_bands", [1, 2, 5])
@pytest.mark.parametrize("bits", [0, 64])
@pytest.mark.parametrize("grid", [0, 256])  # 256: the 528 bricks of the last shape are listed
def test_bricks_at_brick_edges(shape, n_bands, bits, grid):
    rng = np.random.default_rng(sum(shape) + n_bands)
    n = int(np.prod(shape))
    band = rng.integers(0, n_bands, size=shape).astype(np.uint8)
    if n_bands == 2:  # winding regions: long paths through several bricks
        band = (rng.random(shape) < 0.25).astype(np.uint8)
    cc = oracle.components(band, n_bands)
    seeds = rng.choice(n, size=max(1, min(n, n // 300 + 2)), replace=False).astype(np.uint32)
    w = rng.integers(0, 65536, size=shape).astype(np.uint16)
    banner(f"brick edges {shape} bands={n_bands} bits={bits} grid={grid}")
    b, c, q, wd = dev(band), dev(cc.comp), dev(seeds), dev(w)
    prev_e = L.lsrvt_set_vt_engine(L.VT_BRICKS)
    prev_k = L.lsrvt_set_tuning(L.TUNE_KEY_BITS, bits)
    prev_g = L.lsrvt_set_tuning(L.TUNE_BR_GRID, grid)
    try:
        cell = L.lsrvt_vt(b, q)
        r = L.lsrvt_cvt(b, c, q, wd, 3)
    finally:
        L.lsrvt_set_vt_engine(prev_e)
        L.lsrvt_set_tuning(L.TUNE_KEY_BITS, prev_k)
        L.lsrvt_set_tuning(L.TUNE_BR_GRID, prev_g)
    assert np.array_equal(host(cell, np.uint32), oracle.vt(cc.comp, seeds))
    want = oracle.cvt(cc.comp, seeds, w, 3)
    assert np.array_equal(host(r.cell, np.uint32), want.cell)
    assert np.array_equal(host(r.sites, np.uint32), want.sites)
