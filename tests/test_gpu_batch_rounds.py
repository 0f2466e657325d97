"""The update loops of a batch, whose rounds start a workgroup for every brick
of every job or stride over lists of the marked ones, with the reset of a pass
done apart or within its first round: jobs of uneven size, site count and
number of updates (one stops while the others go on, one has none), bit for
bit against the oracle's loop of each job alone."""
import numpy as np
import pytest

import oracle
import paper_2208_06970_amd as L
import synth
from tests.gpu_util import banner, dev, host

pytestmark = pytest.mark.gpu

SPECS = [((16, 16, 16), 1, 2, 3, 64.0), ((17, 33, 31), 2, 4, 5, 20.0), ((5, 40, 18), 3, 3, 0, 30.0),
         ((48, 31, 33), 4, 3, 1, 400.0), ((2, 18, 2200), 5, 3, 2, 60.0)]


@pytest.mark.parametrize("grid", [0, 256])  # 256: below the 313 bricks of all jobs, so they are listed
@pytest.mark.parametrize("reset", [0, 1, 2])
@pytest.mark.parametrize("bits", [0, 64])
def test_batch_rounds_match_oracle(grid, reset, bits):
    jobs, want = [], []
    for shape, seed, n_iso, iters, rho in SPECS:
        f = synth.fourier_field(shape, seed, n_modes=32)
        iso = synth.quantile_isovalues(f, [(i + 1) / (n_iso + 1) for i in range(n_iso)])
        w = synth.gradient_weight(f)
        cc = oracle.components(oracle.bands(f, iso), n_iso + 1)
        seeds = synth.seed_sites(cc.comp, cc.n_comp, w, rho, seed)
        want.append(oracle.cvt(cc.comp, seeds, w, iters))
        jobs.append(L.BatchJob(field=dev(f), iso=iso, seeds=dev(seeds), weights=dev(w), iters=iters,
                               variables=dev(f[None].copy()), cap_comp=int(cc.n_comp)))
    banner(f"batch rounds grid={grid} reset={reset} bits={bits}")
    old = [(k, L.lsrvt_set_tuning(k, v)) for k, v in
           ((L.TUNE_BR_GRID, grid), (L.TUNE_RESET, reset), (L.TUNE_KEY_BITS, bits))]
    try:
        L.lsrvt_batch_run(jobs)
    finally:
        for k, v in old:
            L.lsrvt_set_tuning(k, v)
    for j, r in zip(jobs, want):
        assert j.status == 0
        np.testing.assert_array_equal(host(j.cell, np.uint32), r.cell)
        np.testing.assert_array_equal(host(j.sites, np.uint32)[:len(r.sites)], r.sites)
