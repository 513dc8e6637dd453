"""The tuner of 2D runs with records times what such a run launches: marching
passes at the records and block passes between them."""
import json

import numpy as np
import pytest

from tests.gpu_util import gpu_prs, host, say

pytestmark = pytest.mark.gpu


def _sim(shape, K, f64=False):
    prs = gpu_prs()
    return prs, prs.Sim(prs.make_params(shape, deta=0.1, W0=10.0, diag_every=K,
                                        precision=prs.PRS_F64 if f64 else prs.PRS_F32), seed=5)


@pytest.mark.parametrize("shape,f64", [((256, 192), False), ((301, 257), False), ((512, 512), True)])
@pytest.mark.parametrize("K", [1, 3, 5])
def test_no_pass_longer_than_the_interval(shape, f64, K):
    say("tune with records", shape, f64, K)
    prs, sim = _sim(shape, K, f64)
    prs.prs_autotune(sim.ctx)
    assert sim.time_blocking() <= max(K, 2)
    # the recomputation's passes have no records: not the record passes' tiling
    _, plain = _sim(shape, K, f64)
    assert prs.prs_get_recompute_tiling(sim.ctx) == prs.prs_get_recompute_tiling(plain.ctx)
    # a tuned run is the default one, bit for bit in its fields and counts
    a, b = sim.step_n(23), plain.step_n(23)
    assert [(r["step"], r["links_dir"], r["wall_sites"]) for r in a] == \
           [(r["step"], r["links_dir"], r["wall_sites"]) for r in b]
    for x, y in zip(sim.state(), plain.state()):
        np.testing.assert_array_equal(host(x), host(y))


def test_choices_with_and_without_records_in_one_file(tmp_path):
    say("tune with and without records")
    cache = str(tmp_path / "tune.json")
    prs, rec = _sim((300, 200), 4)
    prs.prs_autotune(rec.ctx, cache)
    first = (rec.tiling(), rec.time_blocking())
    # the only entry serves runs without records too
    _, plain = _sim((300, 200), 0)
    prs.prs_autotune(plain.ctx, cache)
    assert (plain.tiling(), plain.time_blocking()) == first and len(json.load(open(cache))) == 1
    assert prs.prs_tuned_tiling(plain.p, cache) == first[0]
    # ... until these have one of their own, which leaves the first
    prs.prs_autotune(plain.ctx, cache, prs.PRS_TUNE_FORCE)
    second = (plain.tiling(), plain.time_blocking())
    assert len(json.load(open(cache))) == 2
    for K, want in ((0, second), (4, first), (7, first)):
        _, sim = _sim((300, 200), K)
        prs.prs_autotune(sim.ctx, cache)
        assert (sim.tiling(), sim.time_blocking()) == want
        assert prs.prs_tuned_tiling(sim.p, cache) == want[0]
