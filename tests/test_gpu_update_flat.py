"""The site update on volumes of one to seven voxels along an axis (up to six,
the search of the nearest voxel of a cell has a form of its own): rings and
winding regions whose centroids lie outside their cells, near and far, alone
(both entry points) and in the loop, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("edge", [1, 2, 3, 6, 7])
@pytest.mark.parametrize("kind", ["rings", "winding"])
def test_flat_volumes(axis, edge, kind):
    shape = [75, 83]
    shape.insert(axis, edge)
    n = int(np.prod(shape))
    rng = np.random.default_rng(10 * axis + edge)
    if kind == "rings":
        g = np.meshgrid(*[np.arange(k) - k // 2 for k in shape], indexing="ij")
        band = (np.sqrt(sum(c * c for c in g)) / 5).astype(np.uint8) % 3
    else:
        band = (rng.random(shape) < 0.25).astype(np.uint8)
    cc = oracle.components(band, 3)
    seeds = np.unique(np.concatenate([cc.comp_first, rng.choice(n, size=n // 300 + 1)])).astype(np.uint32)
    w = rng.integers(0, 65536, size=shape).astype(np.uint16)
    banner(f"flat {shape} {kind}")
    b, c, q, wd = dev(band), dev(cc.comp), dev(seeds), dev(w)
    cell = oracle.vt(cc.comp, seeds)
    want = oracle.update(cell, seeds, w)[0]
    for run in (L.lsrvt_update, L.lsrvt_update_noalloc):
        got, _ = run(dev(cell), q.clone(), wd)
        assert np.array_equal(host(got, np.uint32), want)
    for engine, bits in ((1, 0), (2, 0), (2, 64)):
        prev_e = L.lsrvt_set_vt_engine(engine)
        prev_k = L.lsrvt_set_tuning(L.TUNE_KEY_BITS, bits)
        try:
            r = L.lsrvt_cvt(b, c, q, wd, 2)
        finally:
            L.lsrvt_set_vt_engine(prev_e)
            L.lsrvt_set_tuning(L.TUNE_KEY_BITS, prev_k)
        full = oracle.cvt(cc.comp, seeds, w, 2)
        assert np.array_equal(host(r.cell, np.uint32), full.cell)
        assert np.array_equal(host(r.sites, np.uint32), full.sites)
