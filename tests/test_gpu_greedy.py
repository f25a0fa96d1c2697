"""The nearest-neighbour tour against the oracle at the edges of its groups of 64
held cities, with candidate lists so short that the fallback chain is used."""
import pytest

from paper_2203_02228_amd import faco as F
from paper_2203_02228_amd import instances as I
from tests.test_gpu_parity import _cmp_setup, _pair, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ls_flags", [0, F.FACO_LS_2OPT])
@pytest.mark.parametrize("n,cl,bl", [(8, 3, 2), (63, 16, 16), (64, 16, 16), (65, 2, 1), (127, 5, 3),
                                     (128, 24, 16), (129, 2, 0), (1025, 16, 64)])
def test_greedy_groups(n, cl, bl, ls_flags):
    say(f"[gpu] greedy n={n} cl={cl} bl={bl} ls={ls_flags}")
    o, g = _pair(I.make_points("cluster16", n, 90 + n), threads=4, n_ants=2, cl_size=cl,
                 bl_size=bl, ls_flags=ls_flags)
    _cmp_setup(o, g)
    g.close()
