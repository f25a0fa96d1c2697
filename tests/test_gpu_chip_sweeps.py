"""Builds whose initial search runs its sweeps as launches over the whole chip
(from 1024 cities on) and inside its own workgroup (below), against the oracle:
initial tour, length and counters, and the first iterations after it."""
import pytest

from paper_2203_02228_amd import faco as F
from paper_2203_02228_amd import instances as I
from tests.test_gpu_parity import _cmp_iter, _cmp_setup, _pair, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tw,ring,n,kind,params", [
    (8, 0, 1023, "uniform", dict()),
    (8, 0, 1024, "uniform", dict()),
    (1, 0, 1025, "cluster16", dict(cl_size=20)),
    (4, 0, 2111, "cluster16", dict(ls_flags=F.FACO_LS_2OPT, cl_size=9)),
    (1, 0, 3001, "uniform", dict(oropt_max_seg=1)),
    (8, 64, 5003, "cluster16", dict()),
    (8, 0, 20011, "uniform", dict(cl_size=5, bl_size=3)),
])
def test_chip_sweeps(tw, ring, n, kind, params):
    say(f"[gpu] chip sweeps tw={tw} ring={ring} n={n} kind={kind} params={params}")
    F.faco_set_team_waves(tw)
    F.faco_set_queue_lds_capacity(ring)
    try:
        o, g = _pair(I.make_points(kind, n, 70 + n), threads=8, n_ants=4, min_new_edges=8, **params)
    finally:
        F.faco_set_queue_lds_capacity(0)
        F.faco_set_team_waves(0)
    _cmp_setup(o, g)
    cnt = F.faco_debug_get(g, F.FACO_DBG_INIT_COUNTERS)
    tk = F.faco_debug_get(g, F.FACO_DBG_INIT_TICKS)
    assert tk[26] == n * cnt[F.CNT_NAMES.index("sweeps")] > 0
    for it in (1, 2):
        o.run(1)
        F.faco_run_iterations(g, 1)
        _cmp_iter(o, g, it)
    g.close()
