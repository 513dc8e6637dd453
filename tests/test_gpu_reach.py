"""Lattices so long and thin that a launch of the usual tiles would hold 2^32
work-items: the library takes other tiles or pass lengths there, and the bits
are those of single steps."""
import pytest

from tests.gpu_util import gpu_prs, say, torch_mod

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2 ** 28 - 1, 1), (1, 7 * 10 ** 8), (1, 1, 6 * 10 ** 8)])
def test_long_thin_lattices(shape):
    say("long", shape)
    torch, prs = torch_mod(), gpu_prs()
    p = prs.make_params(shape, deta=0.1, W0=10.0, diag_every=10)
    many, one = prs.Sim(p, seed=3), prs.Sim(p, seed=3)
    one.set_time_blocking(1)
    one.set_tiling(1, 64, 1)
    for n in (3, 16):
        ra, rb = many.step_n(n), one.step_n(n)
        assert [(r["links_dir"], r["wall_sites"]) for r in ra] == [(r["links_dir"], r["wall_sites"]) for r in rb]
        for a, b in zip(many.state(), one.state()):
            assert torch.equal(a, b), (shape, n)
    many.close()
    one.close()
