"""Line-of-sight passes on volumes short along x and large enough that the bit
planes lie along y or z (more than 6000 tiles along x): the smallest such and
the largest that are not, words and tiles that end inside, at and past the
volume, bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,fill", [
    ((300, 318, 1), 0.3), ((304, 318, 1), 0.05), ((304, 318, 1), 0.3), ((320, 305, 1), 0.3), ((159, 610, 2), 0.3),
    ((24010, 1, 3), 0.05), ((2, 24003, 3), 0.3), ((311, 313, 4), 0.05), ((641, 160, 7), 0.05), ((160, 641, 7), 0.05),
])
def test_los_short_along_x_and_large(shape, fill):
    rng = np.random.default_rng(sum(shape))
    comp = oracle.components((rng.random(shape) < fill).astype(np.uint8), 2).comp
    n = int(np.prod(shape))
    seeds = rng.choice(n, size=n // 20, replace=False).astype(np.uint32)
    w = rng.integers(1, 65536, size=shape).astype(np.uint16)
    banner(f"los short along x {shape} {fill}")
    r = L.lsrvt_los_cvt(dev(comp), dev(seeds), dev(w), 1)
    want = oracle.los_cvt(comp, seeds, w, 1)
    for k in ("cell", "src", "phi"):
        np.testing.assert_array_equal(host(getattr(r.vt, k), np.uint32), getattr(want, k))
    np.testing.assert_array_equal(host(r.vt.dist), want.dist)
    np.testing.assert_array_equal(host(r.site_q), want.site_q)
