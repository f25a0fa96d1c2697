"""Sweeps by a team that gather the touched cities in the queue's LDS ring and
need several passes of it: a ring just above the smallest that is taken as the
list (four times the team's lanes), and ants that touch more cities than it
holds, against the oracle."""
import numpy as np
import pytest

from paper_2203_02228_amd import faco as F
from paper_2203_02228_amd import instances as I
from tests.test_gpu_parity import _cmp_iter, _cmp_setup, _pair, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tw,ring,m", [(4, 1100, 1500), (8, 2100, 2600)])
def test_ring_as_list_in_passes(tw, ring, m):
    n = 20011
    say(f"[gpu] sweep passes tw={tw} ring={ring} m={m}")
    F.faco_set_team_waves(tw)
    F.faco_set_queue_lds_capacity(ring)
    try:
        o, g = _pair(I.make_points("cluster16", n, 31), threads=8, n_ants=3, min_new_edges=m)
    finally:
        F.faco_set_queue_lds_capacity(0)
        F.faco_set_team_waves(0)
    _cmp_setup(o, g)
    for it in (1, 2):
        o.run(1)
        F.faco_run_iterations(g, 1)
        _cmp_iter(o, g, it)
    # cities tested per sweep, on average over each ant's sweeps: above the ring
    tested = F.faco_debug_get(g, F.FACO_DBG_PHASE_TICKS)[:, 26]
    sweeps = F.faco_debug_get(g, F.FACO_DBG_COUNTER_TOTALS)[:, F.CNT_NAMES.index("sweeps")]
    assert np.all(sweeps > 0) and np.any(tested > ring * sweeps), (tested, sweeps)
    assert int(F.faco_debug_get(g, F.FACO_DBG_FAULT)[0]) == 0
    g.close()
