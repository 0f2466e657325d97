"""One site update whose current sites are no voxels of the volume: only the
move's length depends on where a site was, so the moved sites are those of any
other current sites, also where the centroid lies outside its cell and the
nearest voxel is searched (shells: near and far searches).  A site with an
empty cell stays."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radius", [3, 13])
@pytest.mark.parametrize("noalloc", [False, True])
def test_update_from_sites_outside_the_volume(radius, noalloc):
    shape = (43, 40, 45)
    n = int(np.prod(shape))
    z, y, x = np.meshgrid(*[np.arange(k) for k in shape], indexing="ij")
    d = np.sqrt((x - 22) ** 2 + (y - 20) ** 2 + (z - 21) ** 2)
    cell = (np.abs(d - radius) < 1.1).astype(np.uint32)  # cell 1: a hollow shell, cell 0: the rest, cell 2: empty
    w = np.ones(shape, np.uint16)
    want = oracle.update(cell, np.array([0, n // 2, 7], np.uint32), w)[0]
    run = L.lsrvt_update_noalloc if noalloc else L.lsrvt_update
    for old in (n, 0xFFFFFFFF):
        banner(f"update from site {old}: radius {radius} noalloc {noalloc}")
        got, _ = run(dev(cell), dev(np.full(3, old, np.uint32)), dev(w))
        assert host(got, np.uint32).tolist() == [int(want[0]), int(want[1]), old]
