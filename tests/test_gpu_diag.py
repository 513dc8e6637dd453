"""Diagnostics kernels at the values where their fast FP64 forms do not
hold: crossing links without a gradient, sites in the vacuum (V = 0), values
whose products leave FP64's normal range, NaN and inf; and the reduction of
many records in one call.  The fast forms and the sums differ from the
oracle's by rounding: each term is good to about 2^-51, so sums of terms of
one sign to 1e-12."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.gpu_util import assert_stats_match, gpu_prs, params_pair, say, torch_mod

pytestmark = pytest.mark.gpu


def _field(kind, shape, rng):
    n = int(np.prod(shape))
    f = rng.uniform(-1.5, 1.5, n)
    if kind == "no_gradient":          # period-2 stripes: every link crosses, both neighbours equal
        f = np.where(np.arange(n) % 2 == 0, 0.5, -0.5)
    elif kind == "vacuum":             # phi = +-1: V = 0 at wall sites
        f = np.where(f >= 0, 1.0, -1.0)
    elif kind == "tiny":               # products of three factors underflow in float64 fields
        f *= 1e-120
    elif kind == "zeros":
        f[rng.integers(0, n, n // 2)] = 0.0
        f[rng.integers(0, n, n // 4)] = -0.0
    return f


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("shape,tiling", [((128, 10), (4, 8, 1)), ((132, 9), (2, 8, 1)), ((66, 7, 5), (1, 8, 2)),
                                          ((130, 20, 6), (2, 8, 16))])
@pytest.mark.parametrize("kind", ["random", "no_gradient", "vacuum", "tiny", "zeros"])
def test_diagnostics_edge_values(kind, shape, tiling, f64):
    if kind == "tiny" and not f64:
        pytest.skip("1e-120 is not a float32 value")
    say("diag edge", kind, shape, tiling, f64)
    torch, prs = torch_mod(), gpu_prs()
    if f64:
        tiling = (min(tiling[0], 2),) + tiling[1:]
        if tiling[2] == 16:
            tiling = (1,) + tiling[1:]
    gp, op = params_pair(shape, 0.1, diag_every=4, precision=prs.PRS_F64 if f64 else prs.PRS_F32)
    rng = np.random.default_rng(5)
    dt = np.float64 if f64 else np.float32
    phi = _field(kind, shape, rng).astype(dt)
    pi = (0.3 * rng.uniform(-1, 1, phi.size)).astype(dt)
    for T in (1, 2):                       # single-step and multi-step diagnostics
        sim = prs.Sim(gp, phi0=torch.from_numpy(phi).cuda(), dphi0=torch.from_numpy(pi).cuda())
        sim.set_tiling(*tiling)
        sim.set_time_blocking(T)
        ref = O.stats(op, phi.astype(np.float64), pi.astype(np.float64), 0)
        assert_stats_match(sim.wall_stats(), ref, ctx=(kind, "standalone"))
        rec = sim.step_n(2)
        assert len(rec) == 1
        assert_stats_match(rec[0], ref, ctx=(kind, T))


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_diagnostics_nonfinite(bad):
    """Sites with NaN or inf are counted, and the record's sums are those of
    the plain formulas (NaN where they give NaN)."""
    say("diag nonfinite", bad)
    torch, prs = torch_mod(), gpu_prs()
    shape = (128, 8)
    gp, op = params_pair(shape, 0.1)
    phi = np.random.default_rng(7).uniform(-1, 1, 1024).astype(np.float32)
    phi[[3, 500, 1023]] = bad
    pi = np.full(1024, 0.1, np.float32)
    pi[77] = bad
    sim = prs.Sim(gp, phi0=torch.from_numpy(phi).cuda(), dphi0=torch.from_numpy(pi).cuda())
    got = sim.wall_stats()
    ref = O.stats(op, phi.astype(np.float64), pi.astype(np.float64), 0)
    assert got["nonfinite"] == ref["nonfinite"] == 4
    assert got["links_dir"] == ref["links_dir"] and got["wall_sites"] == ref["wall_sites"]
    for key in ("area_density", "gv2"):
        assert np.isnan(got[key]) == np.isnan(ref[key]), key


@pytest.mark.parametrize("shape,tiling,T", [((96, 40), (1, 8, 1), 2), ((64, 24, 20), (1, 8, 8), 2)])
def test_many_records_in_one_call(shape, tiling, T):
    """More records than one reduction launch takes, against the standalone
    diagnostics of the same states."""
    say("many records", shape)
    prs = gpu_prs()
    gp, _ = params_pair(shape, 0.2, diag_every=2)
    steps = 82
    sims = []
    for _ in range(2):
        s = prs.Sim(gp, seed=11)
        s.set_tiling(*tiling)
        s.set_time_blocking(T)
        sims.append(s)
    recs = sims[0].step_n(steps)
    assert [r["step"] for r in recs] == list(range(0, steps, 2))
    for r in recs:
        assert_stats_match(r, sims[1].wall_stats(), ctx=r["step"])
        sims[1].step_n(2, diag=False)
