"""3D LDS passes whose wave holds a whole row (nx of 64 sites a lane: the wave
is a ring, no halo lanes) and the five-step pass of lattices beyond the
last-level cache, against single steps: fields bit for bit, records' counts
exactly and their FP64 sums to the rounding of another order."""
import numpy as np
import pytest

from tests.gpu_util import gpu_prs, host, say

pytestmark = pytest.mark.gpu


def _pair(shape, f64, K=0, beta=0.0):
    prs = gpu_prs()
    p = prs.make_params(shape, deta=0.1, alpha=2.0 if beta else 3.0, beta=beta, m=1.0, W0=10.0, diag_every=K,
                        precision=prs.PRS_F64 if f64 else prs.PRS_F32)
    one, many = prs.Sim(p, seed=4), prs.Sim(p, seed=4)
    one.set_time_blocking(1)
    return one, many


def _same(one, many, what):
    for x, y in zip(one.state(), many.state()):
        np.testing.assert_array_equal(host(x), host(y), err_msg=str(what))


def _records(a, b):
    assert [(r["step"], r["links_dir"], r["wall_sites"]) for r in a] == \
           [(r["step"], r["links_dir"], r["wall_sites"]) for r in b]
    for r, q in zip(a, b):
        for key in ("area_density", "gv2"):
            assert r[key] == pytest.approx(q[key], rel=1e-11)


@pytest.mark.parametrize("vec,ty,f64", [(1, 8, False), (1, 16, False), (1, 32, False), (1, 64, False),
                                        (2, 8, False), (2, 16, False), (2, 32, False), (1, 8, True), (1, 16, True)])
@pytest.mark.parametrize("ny,nz", [(1, 1), (8, 9), (37, 21), (70, 64)])
def test_whole_row_passes(vec, ty, f64, ny, nz):
    say("whole rows", vec, ty, f64, ny, nz)
    one, many = _pair((64 * vec, ny, nz), f64, K=5)
    for T, rows in ((2, 8), (3, 16), (4, 8), (4, 64)):
        many.set_tiling(vec, rows, ty)
        many.set_time_blocking(T)
        for n in (1, 4, 13):
            _records(one.step_n(n), many.step_n(n))
            _same(one, many, (T, rows, n))


# 16 (32) bytes a site and more than the 256 MB last-level cache
@pytest.mark.parametrize("shape,f64,beta", [((250, 274, 281), False, 0.0), ((1186, 25, 640), False, 2.0),
                                            ((128, 1000, 150), False, 0.0), ((131, 270, 271), True, 0.0),
                                            ((64, 23, 6500), True, 0.0)])
def test_five_step_passes(shape, f64, beta):
    say("five steps", shape, f64, beta)
    one, many = _pair(shape, f64, beta=beta)
    for n in (5, 10, 13, 31):
        one.step_n(n)
        many.step_n(n)
        _same(one, many, (shape, n))
    # set to four steps a pass: five between the records all the same
    many.set_tiling(1 if f64 else 2, 16, 16)
    many.set_time_blocking(4)
    one.step_n(21)
    many.step_n(21)
    _same(one, many, (shape, "set"))


def _gradients(shape, f64, nsteps, K, settings):
    from tests.gpu_util import torch_mod
    torch, prs = torch_mod(), gpu_prs()
    p = prs.make_params(shape, deta=0.1, W0=10.0, precision=prs.PRS_F64 if f64 else prs.PRS_F32)
    nb = prs.prs_adjoint_workspace_bytes(p, nsteps, K)
    sim = prs.Sim(p, seed=11)
    if settings is None:
        sim.set_time_blocking(1)
        prs.prs_set_adjoint_time_blocking(sim.ctx, 1)
    elif settings:
        vec, rows, ty, T = settings
        prs.prs_set_adjoint_tiling(sim.ctx, vec, rows, ty)
        prs.prs_set_adjoint_time_blocking(sim.ctx, T)
    work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    g, gd = torch.empty_like(sim.phi_a), torch.empty_like(sim.phi_a)
    loss = prs.prs_adjoint_forward(sim.ctx, nsteps, K, work.data_ptr(), nb)
    gw = prs.prs_adjoint_backward(sim.ctx, work.data_ptr(), nb, g.data_ptr(), gd.data_ptr())
    return loss, gw, host(g).copy(), host(gd).copy()


def _same_gradients(got, want, terms):
    assert got[0] == want[0]
    np.testing.assert_array_equal(got[2], want[2])
    np.testing.assert_array_equal(got[3], want[3])
    # the same FP64 terms of either sign, summed in another order
    assert abs(got[1] - want[1]) <= 1e-12 * max(abs(want[1]), 1e-3 * np.sqrt(terms))


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(64, 9, 8), (128, 37, 21), (37, 30, 50), (202, 20, 33), (1, 2, 3)])
def test_reverse_lds_passes(shape, f64):
    say("reverse", shape, f64)
    nsteps, K = 22, 9
    want = _gradients(shape, f64, nsteps, K, None)
    for ty in (8, 16):
        for vec in (1, 2):
            if shape[0] % vec:
                continue
            for T, rows in ((2, 8), (3, 16), (4, 8)):
                got = _gradients(shape, f64, nsteps, K, (vec, rows, ty, T))
                _same_gradients(got, want, nsteps * want[2].size)


# w, mu and their outputs beyond 150 MB: the stored fields go past the cache
@pytest.mark.parametrize("shape,f64", [((250, 190, 201), False), ((128, 1000, 75), False), ((131, 190, 200), True)])
def test_streamed_adjoint_fields(shape, f64):
    say("streamed", shape, f64)
    nsteps, K = 13, 7
    want = _gradients(shape, f64, nsteps, K, None)
    _same_gradients(_gradients(shape, f64, nsteps, K, ()), want, nsteps * want[2].size)
