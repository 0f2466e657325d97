"""A call whose narrow relaxation keys run out of distance by the library's own
choice: over noise with a site for every component (long winding paths, bricks
relaxed many times) it goes on by levels, also where the sites are too many for
narrow keys, over a wide band with one site beside many it stays with the
relaxation.  Same cells, sites and displacements as with
each schedule asked for, whose parity with the oracle other tests check."""
import numpy as np
import pytest

import paper_2208_06970_amd as L
from tests.gpu_util import banner, torch

pytestmark = pytest.mark.gpu


def _noise(edge, bits):
    t = torch()
    g = t.Generator(device="cuda").manual_seed(3)
    band = t.randint(0, 3, (edge,) * 3, device="cuda", generator=g, dtype=t.uint8)
    cc = L.lsrvt_components(band, 3, cap_comp=1 << bits)
    assert 1 << (bits - 1) < cc.n_comp <= 1 << bits
    return band, cc.comp, cc.comp_first.contiguous()


def _one_beside_many():
    """The site at a corner of 512 x 512 x 24 voxels: up to 1045 hops."""
    t = torch()
    shape = (48, 512, 512)
    band = t.zeros(shape, dtype=t.uint8, device="cuda")
    band[:24] = 1
    cc = L.lsrvt_components(band, 2)
    half = 24 * 512 * 512
    seeds = 2 * t.arange((1 << 21) + 5, device="cuda", dtype=t.int32)  # 22 bits for the ids, 1022 hops
    return band, cc.comp, t.cat([seeds, t.tensor([half], device="cuda", dtype=t.int32)])


@pytest.mark.parametrize("case,engines", [("noise", 1), ("noise, wide keys", 1), ("one beside many", 2)])
def test_after_narrow_keys(case, engines):
    t = torch()
    banner(f"narrow keys run out: {case}")
    # (22 bits for the ids leave 1022 hops, 25 do not fit)
    band, comp, seeds = {"noise": lambda: _noise(256, 22), "noise, wide keys": lambda: _noise(512, 25),
                         "one beside many": _one_beside_many}[case]()
    L.lsrvt_timing_enable(True)
    try:
        L.lsrvt_timing_read()
        got = L.lsrvt_cvt(band, comp, seeds, None, 2)
        cell = L.lsrvt_vt(band, seeds)
        assert L.lsrvt_timing_read()[4] == engines
    finally:
        L.lsrvt_timing_read()
        L.lsrvt_timing_enable(False)
    for engine in (L.VT_LEVELS, L.VT_BRICKS):
        prev = L.lsrvt_set_vt_engine(engine)
        try:
            want = L.lsrvt_cvt(band, comp, seeds, None, 2)
            assert t.equal(L.lsrvt_vt(band, seeds), cell)
        finally:
            L.lsrvt_set_vt_engine(prev)
        assert t.equal(got.cell, want.cell) and t.equal(got.sites, want.sites)
        np.testing.assert_array_equal(got.mean_ds, want.mean_ds)
