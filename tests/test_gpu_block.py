"""2D block passes (several steps with a block of the lattice in registers)
against single steps: the same bits for every block shape's edges -- lattices
narrower than a block, sides that leave ragged blocks, odd widths, one site --
every number of steps a launch takes, both precisions, unit and general
spacing, and in the runs, the ensemble and the adjoint's forward that use
them."""
import numpy as np
import pytest

from tests.gpu_util import gpu_prs, host, say, torch_mod

pytestmark = pytest.mark.gpu


def _pair(shape, f64, dx=1.0, phi0=1.0, beta=0.0, diag_every=0, seed=5):
    prs = gpu_prs()
    p = prs.make_params(shape, deta=0.2 * dx, dx=dx, phi0=phi0, beta=beta, alpha=2.0 if beta else 3.0, m=1.0,
                        W0=10.0, diag_every=diag_every, precision=prs.PRS_F64 if f64 else prs.PRS_F32)
    one, many = prs.Sim(p, seed=seed), prs.Sim(p, seed=seed)
    one.set_time_blocking(1)
    return prs, p, one, many


def _same(one, many, ctx):
    for a, b in zip(one.state(), many.state()):
        np.testing.assert_array_equal(host(a), host(b), err_msg=str(ctx))


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape", [(1, 1), (3, 2), (17, 40), (64, 5), (96, 33), (130, 257), (333, 91), (514, 300),
                                   (1000, 750), (1024, 1024)])
def test_block_passes_match_single_steps(shape, f64):
    say("block", shape, f64)
    prs, _, one, many = _pair(shape, f64)
    steps = list(range(1, 18)) + [31, 33, 50, 100]
    if shape[0] * shape[1] > 1 << 19:
        steps = [1, 2, 5, 8, 11, 13, 16, 17, 40]
    for n in steps:
        one.step_n(n, diag=False)
        many.step_n(n, diag=False)
        _same(one, many, (shape, n))
    assert prs.prs_plan_passes(many.ctx, 100, False)[0] % 2 == 0


@pytest.mark.parametrize("f64", [False, True])
def test_block_passes_general_spacing_and_force(f64):
    say("block general", f64)
    for kw in (dict(dx=0.5), dict(phi0=1.5), dict(beta=2.0)):
        _, _, one, many = _pair((200, 118), f64, **kw)
        for n in (3, 16, 29):
            one.step_n(n, diag=False)
            many.step_n(n, diag=False)
        _same(one, many, kw)


@pytest.mark.parametrize("T,K", [(2, 7), (3, 10), (8, 8), (8, 20), (4, 64), (8, 5)])
def test_runs_with_records(T, K):
    """Records keep their states whatever the passes between them."""
    say("block records", T, K)
    _, _, one, many = _pair((384, 200), False, diag_every=K)
    many.set_time_blocking(T)
    for n in (1, K, 3 * K + 1, 66):
        a, b = one.step_n(n), many.step_n(n)
        assert [r["step"] for r in a] == [r["step"] for r in b]
        assert [r["links_dir"] for r in a] == [r["links_dir"] for r in b]
        assert [r["wall_sites"] for r in a] == [r["wall_sites"] for r in b]
        _same(one, many, (T, K, n))


def test_large_lattice_many_blocks():
    """More blocks than the device holds at once, ragged on both sides."""
    say("block large")
    _, _, one, many = _pair((3002, 2505), False)
    for n in (12, 16, 5):
        one.step_n(n, diag=False)
        many.step_n(n, diag=False)
    _same(one, many, "3002 x 2505")


def test_ensemble_final_state_follows_the_mode():
    """The stream modes' launches differ in number from the persistent
    modes' passes, and with them the buffer of the final field."""
    say("block ensemble")
    torch, prs = torch_mod(), gpu_prs()
    specs = [dict(shape=s, deta=0.25, nsteps=n, diag_every=k, seed=3 + n)
             for s, n, k in (((128, 96), 37, 0), ((64, 64), 20, 6), ((200, 50), 1, 0), ((96, 96), 0, 4))]
    ref = []
    for sp in specs:
        p = prs.make_params(sp["shape"], deta=sp["deta"], diag_every=sp["diag_every"])
        sim = prs.Sim(p, seed=sp["seed"])
        sim.set_time_blocking(1)
        sim.step_n(sp["nsteps"], diag=False)
        ref.append([host(t).copy() for t in sim.state()])
    b = prs.Batch(specs)
    for mode in (prs.PRS_BATCH_STREAMS, prs.PRS_BATCH_PERSISTENT, prs.PRS_BATCH_STREAMS_GRAPH,
                 prs.PRS_BATCH_STREAMS_GRAPH, prs.PRS_BATCH_PERSISTENT_GRAPH, prs.PRS_BATCH_STREAMS):
        b.set_mode(mode)
        b.run()
        torch.cuda.synchronize()
        for r, want in enumerate(ref):
            for got, w in zip(b.final_state(r), want):
                np.testing.assert_array_equal(host(got), w, err_msg=str((mode, r)))
