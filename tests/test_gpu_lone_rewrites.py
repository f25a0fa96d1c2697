"""Rewrites by one-wave ants, which keep 4 chunks of 64 elements in flight up to
256 elements (pairs of a reversal) and 8 beyond: tours whose longest rewrite lies
on either side, against the oracle."""
import pytest

from paper_2203_02228_amd import faco as F
from paper_2203_02228_amd import instances as I
from tests.test_gpu_parity import _cmp_iter, _cmp_setup, _pair, say

pytestmark = pytest.mark.gpu


# a reversal has at most n / 4 pairs, a block move at most n / 2 elements
@pytest.mark.parametrize("n,kind", [(510, "uniform"), (530, "uniform"), (1022, "uniform"),
                                    (1060, "cluster16"), (9001, "cluster16")])
def test_lone_rewrites(n, kind):
    say(f"[gpu] lone rewrites n={n} kind={kind}")
    F.faco_set_team_waves(1)
    try:
        o, g = _pair(I.make_points(kind, n, 40 + n), threads=8, n_ants=6, min_new_edges=30)
    finally:
        F.faco_set_team_waves(0)
    _cmp_setup(o, g)
    for it in (1, 2, 3):
        o.run(1)
        F.faco_run_iterations(g, 1)
        _cmp_iter(o, g, it)
    g.close()
