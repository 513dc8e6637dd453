"""prs_plan_passes takes a const context: threads may ask for plans of one
context side by side, so a call writes nothing to it."""
import ctypes
from concurrent.futures import ThreadPoolExecutor

import pytest

from tests.gpu_util import gpu_prs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(512, 300), (64, 48, 40)])
def test_plans_of_a_fresh_context(shape):
    say("plan", shape)
    prs = gpu_prs()
    sim = prs.Sim(prs.make_params(shape, deta=0.1, W0=10.0, diag_every=10), seed=1)
    # the context begins with its parameters and settings; it is larger than this
    size = 384
    before = ctypes.string_at(sim.ctx, size)
    want = prs.prs_plan_passes(sim.ctx, 95, True)
    assert ctypes.string_at(sim.ctx, size) == before
    with ThreadPoolExecutor(8) as pool:
        plans = list(pool.map(lambda _: prs.prs_plan_passes(sim.ctx, 95, True), range(64)))
    assert plans == [want] * 64
    sim.step_n(20)
    assert prs.prs_plan_passes(sim.ctx, 95, True) == want
