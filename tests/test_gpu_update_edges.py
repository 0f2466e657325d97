"""The site update where its steps change: centroids outside their cells at
distances up to, at and past the near search's cubes (half-width 4), shells
whose nearest voxel is far away, bricks with more cells than the sums' table
holds, weights of zero and the largest weights, in the loop (from the search's
own keys, both schedules and key widths) and alone, bit for bit against the
oracle."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


def _shells(shape, radius):
    """Band 1: a spherical shell of the given radius around the middle; band 0: the rest."""
    z, y, x = np.meshgrid(*[np.arange(n) for n in shape], indexing="ij")
    d = np.sqrt((x - shape[2] // 2) ** 2 + (y - shape[1] // 2) ** 2 + (z - shape[0] // 2) ** 2)
    return (np.abs(d - radius) < 1.1).astype(np.uint8)


@pytest.mark.parametrize("radius", [1.5, 3, 4, 5, 7, 9, 13, 18])
@pytest.mark.parametrize("engine,bits", [(1, 0), (2, 0), (2, 64)])
def test_far_centroids(radius, engine, bits):
    shape = (43, 40, 45)
    band = _shells(shape, radius)
    cc = oracle.components(band, 2)
    flat = band.ravel()
    seeds = np.array([np.flatnonzero(flat == 1)[0], np.flatnonzero(flat == 0)[-1]], dtype=np.uint32)
    w = np.where(band == 1, 65535, 1).astype(np.uint16)
    banner(f"far centroids: radius {radius} engine {engine} bits {bits}")
    b, c, q, wd = dev(band), dev(cc.comp), dev(seeds), dev(w)
    prev_e = L.lsrvt_set_vt_engine(engine)
    prev_k = L.lsrvt_set_tuning(L.TUNE_KEY_BITS, bits)
    try:
        r = L.lsrvt_cvt(b, c, q, wd, 3)
    finally:
        L.lsrvt_set_vt_engine(prev_e)
        L.lsrvt_set_tuning(L.TUNE_KEY_BITS, prev_k)
    want = oracle.cvt(cc.comp, seeds, w, 3)
    assert np.array_equal(host(r.cell, np.uint32), want.cell)
    assert np.array_equal(host(r.sites, np.uint32), want.sites)
    cell = oracle.vt(cc.comp, seeds)
    s2, _ = L.lsrvt_update(dev(cell), q.clone(), wd)
    assert np.array_equal(host(s2, np.uint32), oracle.update(cell, seeds, w)[0])


@pytest.mark.parametrize("per_cell", [1, 2, 5, 600])
@pytest.mark.parametrize("engine", [1, 2])
def test_many_cells_a_brick(per_cell, engine):
    shape = (17, 33, 40)
    n = int(np.prod(shape))
    rng = np.random.default_rng(per_cell)
    band = (rng.random(shape) < 0.3).astype(np.uint8)
    cc = oracle.components(band, 2)
    seeds = rng.choice(n, size=n // per_cell, replace=False).astype(np.uint32)
    w = rng.integers(0, 65536, size=shape).astype(np.uint16)
    w[rng.random(shape) < 0.2] = 0
    w[rng.random(shape) < 0.2] = 65535
    banner(f"cells a brick: {per_cell} voxels a cell, engine {engine}")
    b, c, q, wd = dev(band), dev(cc.comp), dev(seeds), dev(w)
    prev = L.lsrvt_set_vt_engine(engine)
    try:
        r = L.lsrvt_cvt(b, c, q, wd, 2)
        u = L.lsrvt_cvt(b, c, q, None, 2)
    finally:
        L.lsrvt_set_vt_engine(prev)
    for got, want in ((r, oracle.cvt(cc.comp, seeds, w, 2)), (u, oracle.cvt(cc.comp, seeds, None, 2))):
        assert np.array_equal(host(got.cell, np.uint32), want.cell)
        assert np.array_equal(host(got.sites, np.uint32), want.sites)
        assert np.array_equal(got.mean_ds, want.mean_ds) or np.allclose(got.mean_ds, want.mean_ds, rtol=1e-13)
