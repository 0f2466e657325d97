"""The line-of-sight passes at the edges of their tiles (32 x 4 x 4 voxels),
of the cube radii (capped at 31) and of the path walk (32 voxels a launch):
volumes one voxel short of, at and past a tile, thin ones, a large empty one,
and a corridor with more bends than one launch follows, bit for bit against
the oracle (which sums and compares the same float64 values in the same
order)."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


def _match(comp, seeds, w, iters, name):
    banner(f"los edges {name} S={len(seeds)}")
    r = L.lsrvt_los_cvt(dev(comp), dev(seeds), dev(w), iters)
    got = r.vt
    want = oracle.los_cvt(comp, seeds, w, iters)
    for k in ("cell", "src", "phi"):
        np.testing.assert_array_equal(host(getattr(got, k), np.uint32), getattr(want, k))
    np.testing.assert_array_equal(host(got.dist), want.dist)
    np.testing.assert_array_equal(host(r.site_q), want.site_q)


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 5, 31), (4, 4, 32), (5, 3, 33), (9, 4, 65), (40, 7, 1)])
@pytest.mark.parametrize("fill", [0.0, 0.3])
def test_los_at_tile_edges(shape, fill):
    rng = np.random.default_rng(sum(shape))
    comp = oracle.components((rng.random(shape) < fill).astype(np.uint8), 2).comp
    n = int(np.prod(shape))
    seeds = rng.choice(n, size=max(1, n // 60), replace=False).astype(np.uint32)
    _match(comp, seeds, rng.integers(1, 65536, size=shape).astype(np.uint16), 2, f"{shape} {fill}")


def test_los_across_a_large_empty_volume():
    shape = (36, 40, 75)
    comp = np.zeros(shape, np.uint32)
    comp[10:12, 5, 40] = 1  # a few voxels that cast shadows
    seeds = np.array([0, 75 * 40 * 36 - 1, 40 + 75 * (5 + 40 * 10)], np.uint32)
    _match(comp, seeds, np.ones(shape, np.uint16), 1, "empty")


def test_los_along_a_winding_corridor():
    shape = (1, 101, 9)
    band = np.ones(shape, np.uint8)
    band[0, ::2, :] = 0
    for k, y in enumerate(range(1, 101, 2)):
        band[0, y, 8 if k % 2 == 0 else 0] = 0
    comp = oracle.components(band, 2).comp
    _match(comp, np.array([0], np.uint32), np.ones(shape, np.uint16), 0, "corridor")
