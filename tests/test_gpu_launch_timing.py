"""The launches that prs_set_launch_timing brackets are those the benchmark
derives its steps per launch from: every multi-step launch without a record,
whatever its length."""
import pytest

import bench
from tests.gpu_util import gpu_prs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,tiling,T", [((300, 200), (2, 8, 1), 4), ((128, 60, 50), (2, 16, 16), 4),
                                            ((64, 48, 40), (1, 16, 8), 3), ((250, 274, 281), (2, 16, 16), 4)])
def test_steps_of_the_timed_launches(shape, tiling, T):
    say("launch timing", shape, T)
    prs = gpu_prs()
    K, S = 25, 110
    sim = prs.Sim(prs.make_params(shape, deta=0.1, W0=10.0, diag_every=K), seed=1)
    sim.set_tiling(*tiling)
    sim.set_time_blocking(T)
    multi, single = prs.prs_plan_passes(sim.ctx, S, True)
    records = prs.prs_records_in(sim.p, 0, S)
    prs.prs_set_launch_timing(sim.ctx, True)
    prs.prs_get_launch_timing(sim.ctx, reset=True)
    sim.step_n(S)
    _, launches = prs.prs_get_launch_timing(sim.ctx, reset=True)
    assert launches == multi - records
    per = bench.timed_steps_per_launch(S, records, T, single, launches)
    longest = 16 if len(shape) == 2 else 5
    assert 1.0 <= per <= longest
    assert per * launches + records * T + single == S
