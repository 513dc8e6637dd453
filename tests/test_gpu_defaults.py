"""Runs whose settings neither the caller nor the tuner chose: the library
picks tilings and pass lengths by the lattice's size, and the results are the
bits of single steps, whatever it picks -- 3D stretches of every length
between two records, odd and small sides, both precisions and forces, the
ensemble and the adjoint."""
import numpy as np
import pytest

from tests.gpu_util import gpu_prs, host, say, torch_mod

pytestmark = pytest.mark.gpu


def _params(shape, f64, beta=0.0, diag_every=0):
    prs = gpu_prs()
    return prs, prs.make_params(shape, deta=0.1, alpha=2.0 if beta else 3.0, beta=beta, m=1.0, W0=10.0,
                                diag_every=diag_every, precision=prs.PRS_F64 if f64 else prs.PRS_F32)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 3, 7), (64, 64, 64), (33, 50, 21), (130, 61, 40), (200, 120, 90)])
def test_3d_default_runs_match_single_steps(shape, f64):
    say("default 3D", shape, f64)
    for beta, K in ((0.0, 0), (2.0, 0), (0.0, 7), (0.0, 4)):
        prs, p = _params(shape, f64, beta, K)
        one, many = prs.Sim(p, seed=2), prs.Sim(p, seed=2)
        one.set_time_blocking(1)
        assert many.time_blocking() == 1
        for n in (1, 2, 3, 5, 8, 11, 20, 73):
            a, b = one.step_n(n), many.step_n(n)
            assert [(r["step"], r["links_dir"], r["wall_sites"]) for r in a] == \
                   [(r["step"], r["links_dir"], r["wall_sites"]) for r in b]
            for x, y in zip(one.state(), many.state()):
                np.testing.assert_array_equal(host(x), host(y), err_msg=str((shape, f64, beta, K, n)))


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape,nsteps,K", [((96, 70), 37, 8), ((130, 33), 5, 64), ((301, 120), 20, 3),
                                            ((64, 48, 40), 21, 8), ((37, 30, 100), 9, 16), ((128, 64, 96), 30, 7)])
def test_default_adjoint_matches_single_reverse_steps(shape, nsteps, K, f64):
    """Gradient fields bit for bit; dL/dW0 is summed in FP64 from the same
    float32 (float64) terms in another order."""
    say("default adjoint", shape, nsteps, K, f64)
    torch = torch_mod()
    prs, p = _params(shape, f64)
    nb = prs.prs_adjoint_workspace_bytes(p, nsteps, K)
    got = []
    for single in (True, False):
        sim = prs.Sim(p, seed=9)
        if single:
            sim.set_time_blocking(1)
            prs.prs_set_adjoint_time_blocking(sim.ctx, 1)
        work = torch.empty(nb, dtype=torch.uint8, device="cuda")
        g, gd = torch.empty_like(sim.phi_a), torch.empty_like(sim.phi_a)
        loss = prs.prs_adjoint_forward(sim.ctx, nsteps, K, work.data_ptr(), nb)
        gw = prs.prs_adjoint_backward(sim.ctx, work.data_ptr(), nb, g.data_ptr(), gd.data_ptr())
        got.append((loss, gw, host(g).copy(), host(gd).copy()))
    assert got[0][0] == got[1][0]
    np.testing.assert_array_equal(got[0][2], got[1][2])
    np.testing.assert_array_equal(got[0][3], got[1][3])
    # n terms of either sign: rounding of the sums against the terms' size
    terms = nsteps * got[0][2].size
    assert abs(got[0][1] - got[1][1]) <= 1e-12 * max(abs(got[0][1]), 1e-3 * np.sqrt(terms))


def test_default_ensemble_matches_default_runs():
    say("default ensemble")
    prs = gpu_prs()
    specs = [dict(shape=s, deta=0.1, nsteps=n, diag_every=k, seed=n)
             for s, n, k in (((40, 30, 20), 23, 5), ((128, 80), 40, 9), ((64, 64, 32), 12, 0), ((37, 21, 11), 7, 3))]
    b = prs.Batch(specs)
    recs = b.run()
    for r, sp in enumerate(specs):
        p = prs.make_params(sp["shape"], deta=sp["deta"], diag_every=sp["diag_every"])
        sim = prs.Sim(p, seed=sp["seed"])
        own = sim.step_n(sp["nsteps"]) + [sim.wall_stats()]
        for got, want in zip(b.final_state(r), sim.state()):
            np.testing.assert_array_equal(host(got), host(want))
        assert recs[r] == own, r
