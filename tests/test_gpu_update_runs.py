"""The site update on cells that are runs of consecutive voxels: runs that end
at a row's or plane's end lie in two far parts (their nearest voxel is found by
the team's search, over much of the volume), a tile holds more cells than the
table of its sums, and few long ones meet in every tile.  Bit for bit against
the oracle, both entry points."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(300, 257, 1), (300, 1, 257), (1, 300, 257), (190, 200, 2), (3, 130, 140),
                                   (120, 6, 130), (120, 130, 7), (40, 50, 60)])
@pytest.mark.parametrize("run", [2, 61, 350, 10**6])
def test_runs(shape, run):
    n = int(np.prod(shape))
    cell = (np.arange(n) // run).astype(np.uint32).reshape(shape)
    S = int(cell.max()) + 1
    rng = np.random.default_rng(run)
    sites = rng.integers(0, n, size=S).astype(np.uint32)
    w = rng.integers(0, 65536, size=shape).astype(np.uint16)
    for wt in (w, None):
        want, _ = oracle.update(cell, sites, wt)
        for f in (L.lsrvt_update, L.lsrvt_update_noalloc):
            banner(f"runs of {run} in {shape}, weights {wt is not None}, {f.__name__}")
            got, _ = f(dev(cell), dev(sites), None if wt is None else dev(wt))
            assert np.array_equal(host(got, np.uint32), want)
