"""Which cached choices and which candidates the autotuner takes (host logic,
no GPU): an entry that another build of the library wrote is not taken, since a
change of kernels changes what is fastest, and a class of more bricks than the
usual relaxation grids hold also tries the one that covers them."""
import json
import types

import pytest

import paper_2208_06970_amd.autotune as at


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("LSRVT_AUTOTUNE_CACHE", str(path))
    monkeypatch.setattr(at, "_CACHE", None)
    monkeypatch.setattr(at, "_device_name", lambda: "dev")
    return path


def _job(shape, n_sites):
    return types.SimpleNamespace(shape=shape), types.SimpleNamespace(numel=lambda: n_sites)


def test_entries_without_a_library_are_ignored(cache):
    old = "vt:dev:n2^18:vps2^9:bands5"
    cache.write_text(json.dumps({old: {"engine": 1}, "brgrid:" + old: {"grid": 1024},
                                 "statstile:m4:" + old: {"tile": 4}, "batch:dev:jobs": {"streams": 2}}))
    band, sites = _job((64, 64, 64), 512)
    assert at.vt_engine(band, sites, 5, tune=False) is None
    assert at.br_grid(band, sites, 5, tune=False) is None
    assert at.stats_tile((64, 64, 64), 512, 5, 4, None, tune=False) is None


def test_entries_of_another_library_are_ignored(cache, monkeypatch):
    band, sites = _job((64, 64, 64), 512)
    key = at.job_class((64, 64, 64), 512, 5)
    at._store(key, {"engine": 1})
    assert at.vt_engine(band, sites, 5, tune=False) == 1
    other = cache.parent / "liblsrvt.so"
    other.write_bytes(b"another build")
    monkeypatch.setattr(at, "LIB_PATH", str(other))
    monkeypatch.setattr(at, "_BUILD", None)
    assert at.job_class((64, 64, 64), 512, 5) != key
    assert at.vt_engine(band, sites, 5, tune=False) is None


@pytest.mark.parametrize("shape,most", [((64, 64, 64), 8192), ((512, 256, 256), 8192), ((512, 512, 160), 16384),
                                        ((512, 512, 256), 16384), ((512, 512, 257), 8192), ((512, 512, 1024), 8192)])
def test_grids_that_cover_the_bricks_are_tried(cache, monkeypatch, shape, most):
    grids = []
    monkeypatch.setattr(at, "lsrvt_set_tuning", lambda knob, v: grids.append(v) or 0)
    monkeypatch.setattr(at, "lsrvt_set_vt_engine", lambda e: 0)
    monkeypatch.setattr(at, "_time", lambda fn, reps=2: -float(grids[-1]))  # the largest grid is the fastest
    band, sites = _job(shape, 4096)
    assert at.br_grid(band, sites, 5) == most
    assert {1024, 2048, 4096, 8192} <= set(grids)
    assert at.br_grid(band, sites, 5, tune=False) == most
