"""Line-of-sight passes on small volumes that are short along x (whose bit
planes lie along x like the others'; the large ones' lie along y or z): words
and tiles one voxel short of, at and past their ends, bit for bit against the
oracle."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(9, 65, 1), (64, 5, 1), (33, 33, 1), (1, 97, 2), (97, 1, 2), (31, 4, 3), (8, 32, 4),
                                   (5, 63, 7), (63, 5, 7), (6, 7, 7), (7, 33, 8), (2, 2, 1)])
@pytest.mark.parametrize("fill", [0.05, 0.3])
def test_los_short_along_x(shape, fill):
    rng = np.random.default_rng(sum(shape))
    comp = oracle.components((rng.random(shape) < fill).astype(np.uint8), 2).comp
    n = int(np.prod(shape))
    seeds = rng.choice(n, size=max(1, n // 40), replace=False).astype(np.uint32)
    w = rng.integers(1, 65536, size=shape).astype(np.uint16)
    banner(f"los short along x {shape} {fill}")
    r = L.lsrvt_los_cvt(dev(comp), dev(seeds), dev(w), 2)
    want = oracle.los_cvt(comp, seeds, w, 2)
    for k in ("cell", "src", "phi"):
        np.testing.assert_array_equal(host(getattr(r.vt, k), np.uint32), getattr(want, k))
    np.testing.assert_array_equal(host(r.vt.dist), want.dist)
    np.testing.assert_array_equal(host(r.site_q), want.site_q)
