"""Candidate and backup lists, heuristic included, against the oracle: sizes
around the window of labels a query starts from (192) and its buffer (256),
integer grids (massive distance ties), the whole coordinate range, short and
long lists."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2203_02228_amd import faco as F
from paper_2203_02228_amd import instances as I
from tests.test_gpu_parity import say

pytestmark = pytest.mark.gpu


def _grid(side, scale=1):
    return np.array([(x, y) for x in range(side) for y in range(side)], dtype=np.int32) * scale


def _points(kind, n):
    if kind == "grid":
        return _grid(n)
    if kind == "wide grid":
        return _grid(n, 1_500_000)
    if kind == "range":
        rng = np.random.default_rng(n)
        return np.unique(rng.integers(0, 1 << 26, (n, 2)).astype(np.int32), axis=0)
    return I.make_points(kind, n, n)


@pytest.mark.parametrize("kind,n,k,bl", [
    ("grid", 2, 16, 64), ("grid", 9, 5, 3), ("grid", 14, 16, 64), ("grid", 70, 16, 64),
    ("wide grid", 40, 12, 64), ("uniform", 81, 16, 64), ("uniform", 97, 32, 64),
    ("uniform", 192, 16, 64), ("uniform", 193, 2, 0), ("uniform", 257, 16, 64),
    ("cluster16", 5003, 32, 64), ("range", 3000, 16, 64), ("uniform", 20011, 12, 40)])
def test_lists(kind, n, k, bl):
    say(f"[gpu] lists {kind} {n} k={k} bl={bl}")
    xy = _points(kind, n)
    params = dict(n_ants=2, min_new_edges=2, cl_size=k, bl_size=bl)
    g = F.faco_build_instance(xy, **params)
    o = O.Oracle(xy, threads=8, **params)
    cl, b = o.lists()
    assert np.array_equal(F.faco_debug_get(g, F.FACO_DBG_CAND_LISTS), cl)
    assert np.array_equal(F.faco_debug_get(g, F.FACO_DBG_BACKUP_LISTS), b)
    d = np.rint(np.hypot(*(xy[:, None].astype(float) - xy[cl].astype(float)).transpose(2, 0, 1)))
    assert np.array_equal(F.faco_debug_get(g, F.FACO_DBG_HEURISTIC), (1.0 / d).astype(np.float32))
    g.close()


def test_equal_cities_are_refused():
    xy = I.uniform(300, 3)
    xy[299] = xy[17]
    with pytest.raises(F.FacoError) as e:
        F.faco_build_instance(xy, n_ants=2)
    assert e.value.code == F.FACO_EDUP
