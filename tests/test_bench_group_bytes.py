"""The bytes the bench reports for a kernel group: those of its kernel and of what
its launches do besides (CPU)."""
import sys
from pathlib import Path

sys.path.insert(0, str(Path(__file__).resolve().parent.parent))
import bench  # noqa: E402


def test_photon_writes_of_a_merged_step_append_the_leptons():
    st = {"kernel_particles": [1000, 1000, 0, 5000, 0], "event_particles": [300, 40], "n_emit": 4000, "n_pair": 40}
    n_main = [200, 200, 100]
    for merged in (True, False):
        for name in ("count_lepton", "scan", "write_lepton", "count_photon", "write_photon"):
            more = 2 * 40 * (48 + 32) if merged and name == "write_photon" else 0
            assert bench.group_bytes(name, st, n_main, 1, merged=merged) == \
                bench.kernel_bytes(name, st, n_main, 1, merged=merged) + more
