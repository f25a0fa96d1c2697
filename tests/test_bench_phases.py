"""bench.py names an iteration's launches as the library times them: the ants
and the update, which is one launch (CPU only)."""
import bench


def test_phase_names():
    got = bench.phase_means([40.0, 0.0, 0.0, 3.0], [10, 0, 0, 10])
    assert got == {"ants": 4.0, "update": 0.3}
