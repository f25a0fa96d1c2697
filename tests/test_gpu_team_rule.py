"""Waves per ant chosen by the library: lone instances around the ant counts
where the choice changes, and default batches on either side of the batch rule
(few ants, many of even tours, many of uneven tours), against the oracle and
against the same instances run alone."""
import numpy as np
import pytest

from paper_2203_02228_amd import faco as F
from paper_2203_02228_amd import instances as I
from tests.test_gpu_parity import _cmp_iter, _cmp_setup, _pair, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ants,tw", [(1, 8), (256, 8), (257, 4), (2048, 4), (2049, 1)])
def test_lone_instance(ants, tw):
    say(f"[gpu] team rule ants={ants}")
    o, g = _pair(I.uniform(90, 5), threads=8, n_ants=ants, min_new_edges=6)
    assert int(F.faco_debug_get(g, F.FACO_DBG_TEAM_WAVES)[0]) == tw
    _cmp_setup(o, g)
    for it in (1, 2):
        o.run(1)
        F.faco_run_iterations(g, 1)
        _cmp_iter(o, g, it)
    g.close()


@pytest.mark.parametrize("count,lo,hi,ants", [
    (3, 60, 900, 16), (40, 30, 90, 16), (33, 50, 70, 64), (33, 20, 1100, 64)])
def test_default_batch(count, lo, hi, ants):
    say(f"[gpu] batch rule count={count} n={lo}..{hi} ants={ants}")
    sizes = [int(round(lo * (hi / lo) ** (((7 * i) % count) / count) ** 2)) for i in range(count)]
    built = [[F.faco_build_instance(I.uniform(n, 300 + i), n_ants=ants, min_new_edges=5,
                                    cl_size=4 + i % 9, seed=i) for i, n in enumerate(sizes)]
             for _ in range(2)]
    F.faco_run_batch(built[0], 3)
    for a, b in zip(*built):
        F.faco_run_iterations(b, 3)
        ta, la = F.faco_get_best_tour(a)
        tb, lb = F.faco_get_best_tour(b)
        assert la == lb and np.array_equal(ta, tb)
        for what in (F.FACO_DBG_ANT_LENGTHS, F.FACO_DBG_PHEROMONE, F.FACO_DBG_COUNTERS):
            assert np.array_equal(F.faco_debug_get(a, what), F.faco_debug_get(b, what))
        a.close()
        b.close()
