"""3D passes with a spacing and a vacuum value other than 1 (their kernels'
general form): LDS passes of two to five steps and the LDS reverse passes
against single steps, fields and gradients bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import gpu_prs, host, say, torch_mod

pytestmark = pytest.mark.gpu


def _params(shape, f64, dx, phi0, K=0):
    prs = gpu_prs()
    return prs, prs.make_params(shape, deta=0.1 * dx, dx=dx, phi0=phi0, W0=10.0 * dx, diag_every=K,
                                precision=prs.PRS_F64 if f64 else prs.PRS_F32)


def _same(one, many, what):
    for x, y in zip(one.state(), many.state()):
        np.testing.assert_array_equal(host(x), host(y), err_msg=str(what))


@pytest.mark.parametrize("dx,phi0", [(0.5, 1.0), (1.0, 1.5), (2.0, 0.75)])
@pytest.mark.parametrize("vec,ty,f64", [(1, 8, False), (1, 16, False), (1, 32, False), (1, 64, False), (2, 8, False),
                                        (2, 16, False), (2, 32, False), (1, 8, True), (1, 16, True)])
def test_lds_passes(vec, ty, f64, dx, phi0):
    say("spacing", vec, ty, f64, dx, phi0)
    for shape in ((64 * vec, 37, 21), (26 * vec, 30, 50)):
        prs, p = _params(shape, f64, dx, phi0, K=5)
        one, many = prs.Sim(p, seed=4), prs.Sim(p, seed=4)
        one.set_time_blocking(1)
        for T, rows in ((2, 8), (3, 16), (4, 8)):
            many.set_tiling(vec, rows, ty)
            many.set_time_blocking(T)
            for n in (4, 13):
                a, b = one.step_n(n), many.step_n(n)
                assert [(r["step"], r["links_dir"], r["wall_sites"]) for r in a] == \
                       [(r["step"], r["links_dir"], r["wall_sites"]) for r in b]
                for r, q in zip(a, b):
                    for key in ("area_density", "gv2"):
                        assert r[key] == pytest.approx(q[key], rel=1e-11)
                _same(one, many, (shape, T, n))


# more than the 256 MB last-level cache, where passes of five steps are taken
@pytest.mark.parametrize("dx,phi0", [(0.5, 1.5), (1.0, 0.75)])
@pytest.mark.parametrize("shape,f64", [((250, 274, 281), False), ((128, 1000, 150), False), ((131, 270, 271), True)])
def test_five_step_passes(shape, f64, dx, phi0):
    say("spacing, five steps", shape, f64, dx, phi0)
    prs, p = _params(shape, f64, dx, phi0)
    one, many = prs.Sim(p, seed=4), prs.Sim(p, seed=4)
    one.set_time_blocking(1)
    for n in (5, 10, 13):
        one.step_n(n)
        many.step_n(n)
        _same(one, many, (shape, n))


def _gradients(shape, f64, dx, phi0, nsteps, K, settings):
    torch = torch_mod()
    prs, p = _params(shape, f64, dx, phi0)
    sim = prs.Sim(p, seed=11)
    if settings is None:
        sim.set_time_blocking(1)
        prs.prs_set_adjoint_time_blocking(sim.ctx, 1)
    elif settings:
        vec, rows, ty, T = settings
        prs.prs_set_adjoint_tiling(sim.ctx, vec, rows, ty)
        prs.prs_set_adjoint_time_blocking(sim.ctx, T)
    nb = prs.prs_adjoint_workspace_bytes(p, nsteps, K)
    work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    g, gd = torch.empty_like(sim.phi_a), torch.empty_like(sim.phi_a)
    loss, gw = prs.prs_adjoint(sim.ctx, nsteps, K, work.data_ptr(), nb, g.data_ptr(), gd.data_ptr())
    return loss, gw, host(g).copy(), host(gd).copy()


def _same_gradients(got, want, nsteps):
    assert got[0] == want[0]
    np.testing.assert_array_equal(got[2], want[2])
    np.testing.assert_array_equal(got[3], want[3])
    # the same FP64 terms of either sign, summed in another order
    assert abs(got[1] - want[1]) <= 1e-12 * max(abs(want[1]), 1e-3 * np.sqrt(nsteps * want[2].size))


@pytest.mark.parametrize("dx,phi0", [(0.5, 1.5), (2.0, 0.75)])
@pytest.mark.parametrize("shape,f64", [((64, 9, 8), False), ((128, 37, 21), False), ((37, 30, 50), False),
                                       ((202, 20, 33), False), ((64, 9, 8), True), ((37, 30, 50), True)])
def test_lds_reverse_passes(shape, f64, dx, phi0):
    say("spacing, reverse", shape, f64, dx, phi0)
    want = _gradients(shape, f64, dx, phi0, 22, 9, None)
    _same_gradients(_gradients(shape, f64, dx, phi0, 22, 9, ()), want, 22)
    for ty in (8, 16):
        for vec in (1, 2):
            if shape[0] % vec or (f64 and vec > 1):
                continue
            for T, rows in ((2, 8), (3, 16), (4, 8)):
                _same_gradients(_gradients(shape, f64, dx, phi0, 22, 9, (vec, rows, ty, T)), want, 22)


# w, mu and their outputs beyond 150 MB
@pytest.mark.parametrize("shape,f64", [((250, 190, 201), False), ((131, 190, 200), True)])
def test_large_gradients(shape, f64):
    say("spacing, large gradient", shape, f64)
    want = _gradients(shape, f64, 0.5, 1.5, 13, 7, None)
    _same_gradients(_gradients(shape, f64, 0.5, 1.5, 13, 7, ()), want, 13)
