"""Staging rounds of the statistics that fit in LDS and that do not: the sums'
order does not depend on the round, so every output is that of the library's
own choice, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_vars,bins,cov", [(5, 32, True), (18, 32, True), (32, 32, True), (18, 32, False)])
def test_staging_rounds(n_vars, bins, cov):
    shape = (24, 40, 36)  # cells of up to 34560 voxels: several items and rounds, the last ones partial
    rng = np.random.default_rng(n_vars)
    band = (np.arange(shape[0])[:, None, None] + np.zeros(shape) > 7).astype(np.uint8)
    cc = oracle.components(band, 2)
    seeds = np.array([0, 5000, 20000, 34559], np.uint32)
    cell = oracle.vt(cc.comp, seeds)
    x = rng.normal(size=(n_vars,) + shape).astype(np.float32)
    e = np.stack([np.linspace(-3, 3, bins + 1)] * n_vars).astype(np.float32)
    a = (dev(cell), dev(seeds), dev(cc.comp.ravel()[seeds]), dev(cc.comp_band), cc.n_comp, 2, dev(x), dev(e))
    want = None
    for tile in (0, 1, 2, 4):
        banner(f"staging round {tile} vars {n_vars} bins {bins} cov {cov}")
        prev = L.lsrvt_set_tuning(L.TUNE_STATS_TILE, tile)
        try:
            levels = L.lsrvt_aggregate(*a, cov=cov)
        finally:
            L.lsrvt_set_tuning(L.TUNE_STATS_TILE, prev)
        got = [host(getattr(v, k)) for v in levels for k in ("n", "mean", "m2", "vmin", "vmax", "hist", "cov")
               if getattr(v, k) is not None]
        want = want or got
        for p, q in zip(got, want):
            np.testing.assert_array_equal(p, q)
