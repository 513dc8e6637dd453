"""prs_plan_passes counts passes by their steps: a step between two records is
a single-step pass, also where a block pass runs it."""
import pytest

from tests.gpu_util import gpu_prs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(16, 16), (256, 256), (512, 300), (2048, 1024)])
def test_single_steps_between_records(shape, f64):
    say("plan counts", shape, f64)
    prs = gpu_prs()
    p = prs.make_params(shape, deta=0.1, W0=10.0, diag_every=3, precision=prs.PRS_F64 if f64 else prs.PRS_F32)
    sim = prs.Sim(p, seed=1)
    assert sim.time_blocking() == 2
    # ten intervals: a record's pass of two steps, and one step
    assert prs.prs_plan_passes(sim.ctx, 30, True) == (10, 10)
    prs.prs_set_launch_timing(sim.ctx, True)
    prs.prs_get_launch_timing(sim.ctx, reset=True)
    sim.step_n(30)
    assert prs.prs_get_launch_timing(sim.ctx, reset=True)[1] == 0      # none of several steps without a record
