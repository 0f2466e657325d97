"""Seeding with block edges below the largest: rows of a block are read sixteen
voxels wide where that stays inside the volume, so rows end before, at and past
blocks, rows and the volume's last voxel.  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [1, 2, 3, 7, 8, 13, 15, 16])
@pytest.mark.parametrize("shape", [(1, 1, 5), (1, 3, 17), (4, 9, 14), (16, 15, 31), (30, 1, 46), (33, 20, 1)])
def test_rows(block, shape):
    rng = np.random.default_rng(block)
    band = (rng.random(shape) < 0.3).astype(np.uint8)
    cc = oracle.components(band, 2)
    w = rng.integers(0, 65536, size=shape).astype(np.uint16)
    lut = rng.integers(0, 2**32, size=65536, dtype=np.uint64).astype(np.uint32)
    for wt, table, rho in ((None, None, 7), (w, None, 20), (w, lut, 2)):
        banner(f"seed rows: block {block} {shape} rho {rho}")
        got = L.lsrvt_seed(dev(cc.comp), dev(cc.comp_first), cc.n_comp, None if wt is None else dev(wt),
                           None if table is None else dev(table), rho=rho, block=block, seed=5)
        want = oracle.seed_stratified(cc.comp, cc.n_comp, wt, table, rho=rho, block=block, seed=5)
        np.testing.assert_array_equal(host(got, np.uint32), want)
