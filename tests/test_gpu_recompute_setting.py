"""prs_get_recompute_tiling returns the setting the backward's recomputation
runs in: chosen by the lattice's size while nothing is set, the forward's once
that is set, and a reported setting, set, changes no bit."""
import numpy as np
import pytest

from tests.gpu_util import gpu_prs, host, say, torch_mod

pytestmark = pytest.mark.gpu


def _gradient(prs, sim, p):
    torch = torch_mod()
    nb = prs.prs_adjoint_workspace_bytes(p, 20, 9)
    work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    g = torch.empty_like(sim.phi_a)
    sim.set_state(sim.start[0], sim.start[1], 0)
    loss, gw = prs.prs_adjoint(sim.ctx, 20, 9, work.data_ptr(), nb, g.data_ptr(), None)
    return loss, gw, host(g).copy()


@pytest.mark.parametrize("shape,steps", [((96, 70), 8), ((301, 33), 8), ((64, 48, 40), 4), ((37, 30, 50), 4)])
def test_reported_recomputation(shape, steps):
    say("recompute setting", shape)
    prs = gpu_prs()
    p = prs.make_params(shape, deta=0.1, W0=10.0)
    sim = prs.Sim(p, seed=7)
    sim.start = [t.clone() for t in sim.state()]
    rec = prs.prs_get_recompute_tiling(sim.ctx)
    assert rec[3] == steps and rec[1] >= 8
    loss, gw, g = _gradient(prs, sim, p)
    prs.prs_set_recompute_tiling(sim.ctx, *rec)
    assert prs.prs_get_recompute_tiling(sim.ctx) == rec
    again = _gradient(prs, sim, p)
    assert again[:2] == (loss, gw)
    np.testing.assert_array_equal(again[2], g)
    # followed again, and the forward's once set
    prs.prs_set_recompute_tiling(sim.ctx, 1, 1, 1, 0)
    assert prs.prs_get_recompute_tiling(sim.ctx) == rec
    sim.set_tiling(1, 16, 1)
    sim.set_time_blocking(2)
    assert prs.prs_get_recompute_tiling(sim.ctx) == (1, 16, 1, 2)
