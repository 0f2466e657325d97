"""Joint moments with infinite values and NaN: the means of components and bands
are those of all their voxels (infinite with one sign of infinity, NaN with both
or with a NaN), whichever member holds the value, and the centred sums that the
value enters are NaN; the other variable is as without it."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [2, 5, 40])  # members of the component: few, and more than one chunk
@pytest.mark.parametrize("values,mean", [((np.inf,), np.inf), ((-np.inf, -np.inf), -np.inf),
                                         ((np.inf, -np.inf), np.nan), ((np.nan,), np.nan)])
def test_group_means(cells, values, mean):
    shape = (4, 5, 3 * cells)
    comp = np.zeros(shape, np.uint32)
    seeds = np.array([3 * i + 1 for i in range(cells)], dtype=np.uint32)  # every third x of the first row
    cell = oracle.vt(comp, seeds)
    rng = np.random.default_rng(cells)
    x0 = rng.normal(size=(2,) + shape).astype(np.float32)
    for first in {0, cells // 2, cells - len(values)}:
        x = x0.copy()
        for k, v in enumerate(values):  # one a cell, not at its site
            x[0, 3, 4, 3 * ((first + k) % cells)] = v
        banner(f"infinite moments: {cells} cells, {values} from cell {first}")
        got = [L.lsrvt_comoments(dev(cell), dev(seeds), dev(np.zeros(cells, np.uint32)), dev(np.zeros(1, np.uint8)), 1, 1,
                                 dev(v)) for v in (x, x0)]
        for unit in (1, 2):
            a, b = got[0][unit], got[1][unit]
            np.testing.assert_array_equal(host(a.mean)[0, 0], mean)
            assert host(a.mean)[0, 1] == host(b.mean)[0, 1]
            for k in ("m2", "m3", "m4"):
                assert np.isnan(host(getattr(a, k))[0, :-1]).all()  # (0 ..): all entries but (1 .. 1)
                assert host(getattr(a, k))[0, -1] == host(getattr(b, k))[0, -1]
