"""Host code of the library on the CPU, against a stand-in for the HIP runtime
(host_stub.py): what each call enqueues, allocates and launches."""
import pytest

from tests import host_stub


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return host_stub.build_stub(tmp_path_factory.mktemp("stub"))


def test_readback_of_a_capturing_stream_is_refused_before_any_copy(stub):
    """A copy enqueued on a capturing stream becomes a node of the caller's
    graph, and every replay would write to memory that the refused call has
    long given back."""
    got = host_stub.run(stub, """
h = build(60)
whats = range(18)
S.stub_reset()
S.stub_set_capturing(1)
refused = 0
for call in [lambda: F.faco_get_best_tour(h)] + [lambda w=w: F.faco_debug_get(h, w) for w in whats]:
    try:
        call()
    except F.FacoError as e:
        refused += e.code == F.FACO_EDEVICE
copies, ln = S.stub_copies(), S.stub_launch_count()
S.stub_set_capturing(0)
F.faco_get_best_tour(h)
print(json.dumps(dict(refused=refused, copies=copies, launches=ln)))
""")
    assert got == {"refused": 19, "copies": 0, "launches": 0}


def test_noalloc_batch_takes_no_host_memory(stub):
    """Also for an uneven batch at the entry point's limit of 256 instances:
    a failed allocation would leave the C entry point as a C++ exception."""
    got = host_stub.run(stub, """
hs = [build(20 + (37 * i) % 100, ants=4) for i in range(256)]
arr = (ctypes.c_void_p * len(hs))(*[h.h for h in hs])
S.stub_reset()
rc = F.lib().faco_run_batch_noalloc(arr, len(hs), 3, None)
print(json.dumps(dict(rc=rc, news=S.stub_news(), events=S.stub_events(), launches=S.stub_launch_count())))
""")
    assert got == {"rc": 0, "news": 0, "events": 0, "launches": 6}


def test_initial_solution_takes_a_team_whatever_the_ants(stub):
    """One ant on an idle chip; a forced number of waves holds for it too."""
    got = host_stub.run(stub, """
out = []
for tw, n, ants in [(0, 300, 16), (0, 300, 400), (0, 300, 4096), (0, 1500, 400), (1, 300, 16),
                    (4, 1500, 16)]:
    F.faco_set_team_waves(tw)
    S.stub_reset()
    h = build(n, ants=ants)
    one = [L["block"][0] for L in launches() if L["grid"] == [1, 1, 1] and L["block"][0] > 1]
    assert len(set(one)) == 1, one
    out.append(one[0] // 64)
    h.close()
print(json.dumps(out))
""")
    assert got == [8, 8, 8, 8, 1, 4]


WAVES = """
out = []
for n, ants, kw in %s:
    F.faco_set_tour_segments(kw.get("seg", 0))
    h = build(n, ants=ants)
    S.stub_reset()
    F.faco_run_iterations(h, 1)
    L = launches()[0]
    assert L["grid"][0] == ants and L["lds"] <= 160 * 1024
    assert int(F.faco_debug_get(h, F.FACO_DBG_TEAM_WAVES)[0]) * 64 == L["block"][0]
    out.append(L["block"][0] // 64)
    h.close()
print(json.dumps(out))
"""


def _waves(stub, cases):
    got = host_stub.run(stub, WAVES % repr([c[:3] for c in cases]))
    assert got == [c[3] for c in cases], list(zip(cases, got))


def test_waves_of_segment_list_ants(stub):
    """Teams up to 512 ants; beyond, lone waves while a CU's LDS holds two ants,
    else teams of 8 (one ant a CU either way)."""
    seg = dict(seg=2)
    _waves(stub, [(300, 256, seg, 8), (300, 257, seg, 4), (300, 512, seg, 4),
                  (300, 513, seg, 1), (300, 4096, seg, 1), (3000, 600, seg, 1),
                  (10000, 600, seg, 1), (14000, 600, seg, 8)])


def test_waves_of_ants_by_lds(stub):
    """Long tours: LDS holds one 4-wave team a CU from about 16 300 cities on
    (with the default queue), so the ants take teams of 8 at any number."""
    flat = {}
    _waves(stub, [(16200, 256, flat, 8), (16200, 300, flat, 4), (16400, 300, flat, 8),
                  (4000, 2048, flat, 4), (4000, 2049, flat, 1), (17000, 2049, flat, 8),
                  (30000, 300, flat, 8)])


def test_workers_of_persistent_batches(stub):
    """One wave a SIMD, and two with 4-wave teams beyond 6 ants a CU (256 CUs,
    room for 8 workgroups on each)."""
    got = host_stub.run(stub, """
out = []
for tw, apb, count, ants in [(1, 1, 16, 256), (1, 1, 10, 64), (1, 2, 16, 256), (1, 4, 16, 256),
                             (4, 1, 6, 256), (4, 1, 7, 256), (4, 1, 3, 64), (8, 1, 16, 64)]:
    F.faco_set_batch_config(persistent=1, team_waves=tw, ants_per_block=apb,
                            queue_lds_capacity=64)
    hs = [build(40, ants=ants) for _ in range(count)]
    S.stub_reset()
    F.faco_run_batch(hs, 3)
    (L,) = launches()
    assert L["block"][0] == 64 * max(tw, apb)
    out.append(L["grid"][0])
print(json.dumps(out))
""")
    assert got == [1024, 640, 512, 256, 256, 512, 192, 256]


def test_events_reserved_for_timed_iterations(stub):
    """Two events for each of an iteration's two launches, and none made while
    the reserved iterations are enqueued."""
    got = host_stub.run(stub, """
h = build(60)
S.stub_reset()
F.faco_set_timing(h, True, reserve_iterations=10)
made = S.stub_events()
F.faco_run_iterations(h, 10)
print(json.dumps([made, S.stub_events() - made]))
""")
    assert got == [40, 0]


def test_waves_of_default_batches(stub):
    """Few ants 8, up to 2048 4; beyond, 1 for even tours and 4 where the mean
    length is below half the longest; 8 where LDS holds one 4-wave team a CU."""
    got = host_stub.run(stub, """
out = []
for sizes, ants in [([60, 500, 900], 16), ([60] * 4, 64), ([60] * 5, 64), ([60] * 32, 64),
                    ([60] * 33, 64), ([200] + [98] * 32, 64), ([200] + [96] * 32, 64),
                    ([16200, 50, 50], 100), ([16400, 50, 50], 100)]:
    hs = [build(n, ants=ants) for n in sizes]
    S.stub_reset()
    F.faco_run_batch(hs, 1)
    L = launches()[0]
    assert L["grid"][0] == ants * len(sizes) and L["lds"] <= 160 * 1024
    out.append(L["block"][0] // 64)
    for h in hs:
        h.close()
print(json.dumps(out))
""")
    assert got == [8, 8, 4, 4, 1, 1, 4, 4, 8]


def test_blocks_of_the_update(stub):
    """A block per 256 slots and per 256 positions, at most 512 and 128 while a
    thread has up to 8 slots and 4 positions, then up to 1024 and 256."""
    got = host_stub.run(stub, """
out = []
for n, k in [(300, 5), (8192, 16), (8193, 16), (33000, 4), (70000, 16), (150000, 16)]:
    h = build(n, ants=2, k=k)
    S.stub_reset()
    F.faco_run_iterations(h, 1)
    out.append(launches()[1]["grid"][0])
    h.close()
print(json.dumps(out))
""")
    assert got == [10 + 2, 512 + 32, 512 + 33, 512 + 128, 546 + 128, 1024 + 146]
