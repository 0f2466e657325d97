"""Joint moments at the edges of the tiled contraction: every split of the
pair tiles over the waves (by the number of variables), cells at and across
the items' length, cells shorter than a step of four voxels, and groups below,
at and above the length of a merge chunk, against the oracle's direct float64
sums.  Tolerance as in test_gpu_moments: a sum of n <= 2^14 products of
float64 offsets errs by less than n 2^-53 of the sum of its terms' sizes, the
shifts to a group's mean add as much again, so 1e-8 of the entry's natural
scale n sigma_i sigma_j ... holds with room."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host
from tests.test_gpu_moments import _check, _units

pytestmark = pytest.mark.gpu
ITEM = 2048  # voxels of an item of the cell sums


def _strip(lengths, shape, seed):
    """A volume whose cells are runs of the given lengths in linear order, one site at the first voxel of each; a
    length of 0 is an empty cell."""
    n = int(np.prod(shape))
    cell = np.full(n, oracle.NONE_ID, dtype=np.uint32)
    sites, at = [], 0
    for s, k in enumerate(lengths):
        sites.append(min(at, n - 1))
        cell[at:at + k] = s
        at += k
    assert at <= n
    return cell.reshape(shape), np.array(sites, dtype=np.uint32)


@pytest.mark.parametrize("m", [1, 5, 9, 10, 15, 17, 18])
def test_tiles_items_and_chunks(m):
    shape = (19, 23, 29)
    rng = np.random.default_rng(m)
    lengths = [1, 3, 4, 5, 63, 64, 65, 0, ITEM - 1, ITEM, ITEM + 1, 2 * ITEM + 7] + [2] * 60
    cell, sites = _strip(lengths, shape, m)
    S = len(lengths)
    # components of 1, 2, 16, 17 and the rest of the cells, in three bands
    counts = [1, 2, 16, 17, S - 36]
    site_comp = np.repeat(np.arange(5), counts).astype(np.uint32)
    comp_band = np.array([0, 0, 1, 2, 2], dtype=np.uint8)
    x = (rng.normal(size=(m,) + shape) + 3.0 * rng.random((m, 1, 1, 1))).astype(np.float32)
    x[0] = x[0] ** 3
    banner(f"moment tiles: m={m}")
    got = L.lsrvt_comoments(dev(cell), dev(sites), dev(site_comp), dev(comp_band), 5, 3, dev(x))
    units = _units(cell, site_comp, comp_band.astype(np.uint32))
    for name, g, u, k in zip(("cell", "comp", "band"), got, units, (S, 5, 3)):
        _check(name, g, oracle.comoments(u, k, x), m)
    assert int(host(got[0].n)[7]) == 0
