"""The exact and the float64 merges at the edges of their kernels: components of
32 and 33 cells (one thread or a workgroup), of more cells than a workgroup's
lanes take in one step (2048), bands of one component, of 33 and of thousands,
empty cells among them; against the oracle's direct FP64 statistics with the
tolerances of test_gpu_stats."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host
from tests.test_gpu_stats import _check_level
from tests.test_gpu_stats_modes import _strip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,bins", [(1, 0), (3, 16), (9, 32)])
def test_merges_of_many_members(m, bins):
    rng = np.random.default_rng(m)
    groups = [1, 32, 33, 255, 257, 2049, 4100] + [1] * 9000  # cells of each component
    lengths = rng.integers(1, 5, size=sum(groups))
    lengths[rng.integers(0, len(lengths), size=200)] = 0
    lengths[-1] = 3
    shape = (3, 130, 160)
    cell, sites = _strip(lengths.tolist(), shape)
    site_comp = np.repeat(np.arange(len(groups)), groups).astype(np.uint32)
    C, S = len(groups), len(lengths)
    band_of = np.full(C, 2, np.uint8)
    band_of[0], band_of[1:34], band_of[-1] = 0, 1, 3
    x = (rng.normal(size=(m,) + shape) + 3.0).astype(np.float32)
    edges = np.stack([np.linspace(v.min(), v.max(), bins + 1) for v in x]).astype(np.float32) if bins else None
    banner(f"merges m={m} bins={bins}")
    got = L.lsrvt_aggregate(dev(cell), dev(sites), dev(site_comp), dev(band_of), C, 4, dev(x),
                            None if edges is None else dev(edges), cov=True)
    none = cell == oracle.NONE_ID
    comp = np.where(none, oracle.NONE_ID, site_comp[np.minimum(cell.astype(np.int64), S - 1)]).astype(np.uint32)
    band = np.where(none, oracle.NONE_ID, band_of.astype(np.uint32)[np.minimum(comp, C - 1)]).astype(np.uint32)
    _check_level("comp", got[1], oracle.stats(comp, C, x, edges, True), m)
    _check_level("band", got[2], oracle.stats(band, 4, x, edges, True), m)
