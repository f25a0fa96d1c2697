"""The local search run by every wave of a team, at the sizes where its
branches change, against the oracle (bit for bit).

Tours of more than 16384 cities need several passes of a sweep's city list;
long tours make reversals and block moves of every share size (one chunk per
wave, four, sixteen; a block of up to 128 cities is one wave's alone); lists of
more than 16 candidates are evaluated by two parts of 32 lanes instead of four
of 16; tours of fewer than 7 cities are shorter than the neighbourhood an
evaluation reads; a small LDS ring takes the sweep's small city list."""
import pytest

from paper_2203_02228_amd import faco as F
from paper_2203_02228_amd import instances as I
from tests.test_gpu_parity import _cmp_iter, _cmp_setup, _pair, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tw,ring,n,kind,iters,params", [
    (8, 0, 4, "uniform", 3, dict(n_ants=3, min_new_edges=2)),
    (4, 0, 6, "uniform", 3, dict(n_ants=3, min_new_edges=2)),
    (8, 0, 7, "uniform", 3, dict(n_ants=3, min_new_edges=3, cl_size=3, bl_size=2)),
    (8, 0, 2049, "cluster16", 3, dict(n_ants=5, min_new_edges=60, cl_size=17)),
    (4, 0, 3001, "uniform", 3, dict(n_ants=4, min_new_edges=50, cl_size=32, bl_size=8)),
    (8, 300, 5003, "cluster16", 3, dict(n_ants=4, min_new_edges=40)),
    (8, 0, 17011, "uniform", 2, dict(n_ants=6, min_new_edges=200)),
    (4, 0, 20011, "cluster16", 2, dict(n_ants=4, min_new_edges=64, cl_size=10)),
])
def test_team_search(tw, ring, n, kind, iters, params):
    say(f"[gpu] team search tw={tw} ring={ring} n={n} kind={kind} params={params}")
    F.faco_set_team_waves(tw)
    F.faco_set_queue_lds_capacity(ring)
    try:
        o, g = _pair(I.make_points(kind, n, 900 + n), threads=8, **params)
    finally:
        F.faco_set_queue_lds_capacity(0)
        F.faco_set_team_waves(0)
    _cmp_setup(o, g)
    for it in range(1, iters + 1):
        o.run(1)
        F.faco_run_iterations(g, 1)
        _cmp_iter(o, g, it)
    assert int(F.faco_debug_get(g, F.FACO_DBG_FAULT)[0]) == 0
    g.close()
