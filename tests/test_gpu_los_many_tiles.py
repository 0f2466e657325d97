"""Line-of-sight pass with more tiles than one run of the grid's x covers
(2^22): a slice of 16500 x 32600 voxels of which only three boxes belong to
components, one in the first tile, one across the end of the run and one in the
last tile.  The boxes' paths do not leave them, so they are those of the boxes
cut out (order of the voxel indices and so the ties included)."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
from tests.gpu_util import banner, host, torch

pytestmark = pytest.mark.gpu

NY, NX = 16500, 32600
NONE = 0xFFFFFFFF


def test_los_past_one_run_of_tiles():
    t = torch()
    h, w = 9, 70
    words = -(-NX // 32)
    row = 4 * ((1 << 22) // words)  # rows of the tile that ends the run
    assert words * -(-NY // 4) > 1 << 22 and 0 < row - 4 and row + h < NY
    x1 = 32 * ((1 << 22) % words) - w // 2  # the run ends inside the box
    boxes = [(0, 0), (row - 2, x1), (NY - h, NX - w)]
    comp = t.full((1, NY, NX), -1, dtype=t.int32, device="cuda")
    rng = np.random.default_rng(4)
    cut, site_q, anchor, own = [], [], [], []
    for k, (y, x) in enumerate(boxes):
        c = oracle.components((rng.random((1, h, w)) < 0.2).astype(np.uint8), 2).comp
        a = rng.choice(h * w, size=6, replace=False)
        ax, ay = a % w, a // w
        cut.append(oracle.los_vt(c, np.stack([256 * ax, 256 * ay, 0 * ax], 1).astype(np.int32), a.astype(np.uint32)))
        comp[0, y:y + h, x:x + w] = t.from_numpy((c[0] + 1000 * k).astype(np.int32)).cuda()
        site_q.append(np.stack([256 * (ax + x), 256 * (ay + y), 0 * ax], 1))
        anchor.append((ax + x) + NX * (ay + y))
        own.append(len(anchor[0]) * k)
    banner("los on 16500 x 32600 voxels")
    q = t.from_numpy(np.concatenate(site_q).astype(np.int32)).cuda()
    r = L.lsrvt_los_vt(comp, q, t.from_numpy(np.concatenate(anchor).astype(np.int32)).cuda(), ws=L.Workspace())

    def placed(v, y, x):  # voxel indices of a box as indices of the volume
        u = np.where(v == NONE, 0, v).astype(np.int64)
        return np.where(v == NONE, NONE, (u % w + x) + NX * (u // w + y)).astype(np.uint32)

    for (y, x), s0, want in zip(boxes, own, cut):
        at = (0, slice(y, y + h), slice(x, x + w))
        np.testing.assert_array_equal(host(r.dist[at].contiguous()), want.dist[0])
        cell = np.where(want.cell == NONE, NONE, want.cell + s0).astype(np.uint32)
        np.testing.assert_array_equal(host(r.cell[at].contiguous(), np.uint32), cell[0])
        np.testing.assert_array_equal(host(r.phi[at].contiguous(), np.uint32), placed(want.phi, y, x)[0])
        seen = (want.src != NONE) & (want.src >= L.LOS_SITE)
        src = np.where(seen, want.src + s0, placed(np.where(seen, 0, want.src), y, x)).astype(np.uint32)
        np.testing.assert_array_equal(host(r.src[at].contiguous(), np.uint32), src[0])
    # nothing else has a path
    assert int((r.cell != -1).sum()) == int(sum((c.cell != NONE).sum() for c in cut))
    del r, comp
    t.cuda.empty_cache()
