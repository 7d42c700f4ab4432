"""Host model of the event log's pool (CPU): ``event_log_pool_model.cpp`` runs
the waves of random launches on one pool with the sizes and the rule of
csrc/event_log.h, reads their logs in the tiles of ``k_replay_events``, and
requires that a pool of exactly the reported need never runs out, that waves
without records need nothing, and that a launch which fits a pool that could not
grow runs out at most once.
"""
import subprocess
from pathlib import Path

HERE = Path(__file__).resolve().parent


def test_event_log_pool_model(tmp_path):
    exe = tmp_path / "event_log_pool_model"
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wno-unknown-pragmas",
                    str(HERE / "event_log_pool_model.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), "300"], capture_output=True, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("0 mistakes, 0 exact pools ran out")
