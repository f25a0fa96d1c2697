"""The iteration's update in one launch: rows padded past lists that are not a
multiple of four, sources taken from the global best and from the iteration
best, tours with several slots per thread (n k > 262144) and several positions
per thread (n > 65536), a lone instance and the same in a batch, against the
oracle."""
import numpy as np
import pytest

from paper_2203_02228_amd import faco as F
from paper_2203_02228_amd import instances as I
from tests.test_gpu_parity import _cmp_iter, _pair, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,p_gb,ants,iters", [
    (33, 5, 1.0, 3, 6), (1500, 2, 0.5, 5, 5), (20011, 14, 0.5, 3, 4), (70001, 6, 0.7, 2, 3)])
def test_update(n, k, p_gb, ants, iters):
    say(f"[gpu] update n={n} k={k} p_source_gbest={p_gb}")
    xy = I.make_points("uniform", n, n)
    params = dict(n_ants=ants, min_new_edges=12, cl_size=k, p_source_gbest=p_gb, rho=0.7, seed=n)
    o, g = _pair(xy, threads=8, **params)
    b = F.faco_build_instance(xy, **params)
    other = F.faco_build_instance(I.uniform(50, 1), n_ants=2, min_new_edges=4)
    for it in range(1, iters + 1):
        o.run(1)
        F.faco_run_iterations(g, 1)
        _cmp_iter(o, g, it)
    F.faco_run_batch([b, other], iters)
    for what in (F.FACO_DBG_PHEROMONE, F.FACO_DBG_SOURCE, F.FACO_DBG_LIMITS, F.FACO_DBG_INFO):
        assert np.array_equal(F.faco_debug_get(b, what), F.faco_debug_get(g, what))
    for h in (g, b, other):
        h.close()
