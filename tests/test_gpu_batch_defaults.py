"""Ensemble members whose settings were not set: short tiles in the stream
modes and on small lattices, taller ones in the persistent modes, and in every
mode the bits of the member run alone with the tiling the ensemble reports."""
import numpy as np
import pytest

from tests.gpu_util import gpu_prs, host, say

pytestmark = pytest.mark.gpu

SPECS = [dict(shape=s, deta=0.1, nsteps=n, diag_every=k, seed=i)
         for i, (s, n, k) in enumerate([((64, 64), 30, 8), ((768, 512), 21, 10), ((1023, 301), 12, 5),
                                        ((24, 24, 24), 14, 5), ((128, 96, 64), 13, 6), ((101, 77, 31), 9, 0)])]


def alone(prs, sp, tiling, T):
    sim = prs.Sim(prs.make_params(sp["shape"], deta=sp["deta"], diag_every=sp["diag_every"]), seed=sp["seed"])
    sim.set_time_blocking(1)
    sim.set_tiling(*tiling)
    sim.set_time_blocking(T)
    return sim.step_n(sp["nsteps"]) + [sim.wall_stats()], [host(x).copy() for x in sim.state()]


@pytest.mark.parametrize("modes", [(1,), (4, 1, 3, 0, 2, 4)])
def test_default_tilings_by_mode(modes):
    say("batch defaults", modes)
    prs = gpu_prs()
    b = prs.Batch(SPECS)
    for mode in modes:
        b.set_mode(mode)
        recs = b.run()
        for r, sp in enumerate(SPECS):
            (vec, rows, ty), T = b.tiling(r)
            large = np.prod(sp["shape"]) > 2 ** 17
            if mode in (0, 1, 2) and large:
                assert rows == (16 if len(sp["shape"]) == 2 else 32), (mode, sp["shape"])
            else:
                assert rows < 16, (mode, sp["shape"])
            want, state = alone(prs, sp, (vec, rows, ty), T)
            for x, y in zip(b.final_state(r), state):
                np.testing.assert_array_equal(host(x), y, err_msg=str((mode, sp["shape"])))
            assert recs[r] == want[-len(recs[r]):], (mode, sp["shape"])
    b.close()


def test_tuned_persistent_settings_stay():
    """The ensemble tuner starts from the mode's tiling, and what it keeps
    counts as set in every mode."""
    say("batch defaults, tuner")
    prs = gpu_prs()
    b = prs.Batch(SPECS[1:3])
    b.set_mode(1)
    before = [b.tiling(r) for r in range(2)]
    prs.prs_batch_autotune(b.b)
    after = [b.tiling(r) for r in range(2)]
    b.set_mode(4)
    for r in range(2):
        assert after[r][0][1] % before[r][0][1] == 0
        if after[r] != before[r]:
            assert b.tiling(r) == after[r]
    b.close()
