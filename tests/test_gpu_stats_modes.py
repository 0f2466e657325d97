"""Statistics at the edges of the cell kernels: every way of taking the
products (squares only; up to 4, 8 and 16 variables; 17 to 20; 21 to 32), cells
at the steps of the small-cell path (16, 32, 64 and 256 voxels) and of the
items (4096), a cell of more than 32 items, and infinite values, against the
oracle's direct FP64 statistics.  Tolerances as in test_gpu_stats: the sums
are float64, so the float32 rounding of the outputs is all that they use."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host
from tests.test_gpu_stats import _check_level

pytestmark = pytest.mark.gpu


def _strip(lengths, shape):
    n = int(np.prod(shape))
    cell = np.full(n, oracle.NONE_ID, dtype=np.uint32)
    sites, at = [], 0
    for s, k in enumerate(lengths):
        sites.append(min(at, n - 1))
        cell[at:at + k] = s
        at += k
    assert at <= n
    return cell.reshape(shape), np.array(sites, dtype=np.uint32)


LENGTHS = [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 0, 255, 256, 257, 4095, 4096, 4097, 33 * 4096 + 5]
COMP = np.repeat(np.arange(4), [1, 7, 9, 2]).astype(np.uint32)
BAND = np.array([0, 0, 1, 1], dtype=np.uint8)


@pytest.mark.parametrize("m,bins,cov", [
    (1, 16, True), (4, 32, True), (5, 0, True), (8, 32, True), (9, 8, True), (16, 32, True), (17, 32, True),
    (20, 5, True), (21, 32, True), (32, 4, True), (1, 16, False), (4, 0, False), (7, 32, False), (20, 32, False),
    (32, 8, False),
])
def test_every_product_mode(m, bins, cov):
    shape = (37, 61, 70)
    rng = np.random.default_rng(100 * m + bins)
    cell, sites = _strip(LENGTHS, shape)
    x = (rng.normal(size=(m,) + shape) * (1 + np.arange(m))[:, None, None, None] + 2.0).astype(np.float32)
    edges = None
    if bins:
        edges = np.stack([np.linspace(v.min(), v.max(), bins + 1) for v in x]).astype(np.float32)
    site_comp = np.concatenate([COMP[:len(LENGTHS) - 1], [3]]).astype(np.uint32)
    S = len(LENGTHS)
    banner(f"product modes: m={m} bins={bins} cov={cov}")
    got = L.lsrvt_aggregate(dev(cell), dev(sites), dev(site_comp), dev(BAND), 4, 2, dev(x),
                            None if edges is None else dev(edges), cov=cov)
    c = cell.astype(np.int64)
    comp = np.where(cell == oracle.NONE_ID, oracle.NONE_ID, site_comp[np.minimum(c, S - 1)]).astype(np.uint32)
    band = np.where(cell == oracle.NONE_ID, oracle.NONE_ID, BAND.astype(np.uint32)[np.minimum(comp, 3)]).astype(np.uint32)
    _check_level("cell", got[0], oracle.stats(cell, S, x, edges, cov), m)
    _check_level("comp", got[1], oracle.stats(comp, 4, x, edges, cov), m)
    _check_level("band", got[2], oracle.stats(band, 2, x, edges, cov), m)


@pytest.mark.parametrize("m,cov", [(3, True), (18, True), (24, True), (3, False)])
def test_infinite_values_stay_in_their_variable(m, cov):
    """An infinity leaves its variable's mean without a number in the cells that hold it, small and large, and every
    other variable as it is without the infinity."""
    shape = (10, 30, 70)
    rng = np.random.default_rng(m)
    cell, sites = _strip([40, 300, 9000, 50], shape)
    x = rng.normal(size=(m,) + shape).astype(np.float32)
    y = x.copy()
    for v in (7, 100, 5000):
        y.reshape(m, -1)[1, v] = np.inf
    args = (dev(cell), dev(sites), dev(np.zeros(4, np.uint32)), dev(np.zeros(1, np.uint8)), 1, 1)
    banner(f"infinities: m={m} cov={cov}")
    a = L.lsrvt_aggregate(*args, dev(x), None, cov=cov)[0]
    b = L.lsrvt_aggregate(*args, dev(y), None, cov=cov)[0]
    keep = [j for j in range(m) if j != 1]
    for k in ("mean", "m2", "vmin", "vmax"):
        assert np.array_equal(host(getattr(a, k))[:, keep], host(getattr(b, k))[:, keep]), k
    assert np.all(np.isnan(host(b.mean)[:3, 1])) and np.all(np.isnan(host(b.m2)[:3, 1]))
    assert np.all(host(b.vmax)[:3, 1] == np.inf)
    assert np.array_equal(host(a.mean)[3], host(b.mean)[3])
