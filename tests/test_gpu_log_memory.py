"""Device memory of the event log: a step takes what the waves with events need,
however many waves its launch has, and a pool that cannot grow stays, so that
launches that fit it are still replayed.  In a process of its own, since the
log's pool lives as long as the process."""
import json
import os
import subprocess
import sys
from pathlib import Path

import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu

CHILD = r"""
import json, os, sys
import torch
import paper_2409_17299_amd as sf

N, MIB = 1_100_000, 1 << 20   # four waves per SIMD: 4096 waves on 256 CUs, half a GiB of log blocks
g = torch.Generator(device="cuda"); g.manual_seed(3)
u = torch.rand(N, dtype=torch.float64, device="cuda", generator=g)
tabs, cfg = sf.Tables(), sf.step_cfg(pair=False, push=False)
main = [sf.Store.empty(n, torch.float32, photon=s == 2) for s, n in enumerate((N, 1, 1))]
zero = torch.zeros(N, device="cuda")
bz = torch.zeros(N, device="cuda")
fields = [sf.Fields(zero, zero, zero, zero, zero, bz, stride=1) for _ in range(3)]
app = [sf.AppendBuffer(4 * N if s == 2 else 1, torch.float32) for s in range(3)]

def step(emitters):
    e = main[0]
    e.px[:], e.py[:], e.pz[:], e.w[:], e.tau[:] = 2000.0, 0.0, 0.0, 1.0, -torch.log(u)
    e.id[:] = torch.arange(N, device="cuda"); e.count = N
    bz.zero_(); bz[:emitters] = 1e-3
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    _, st = sf.step(tabs, main, fields, app, 5e4, 5, 1, cfg)
    torch.cuda.synchronize()
    return dict(taken=before - torch.cuda.mem_get_info()[0], replays=st.log_replays, reruns=st.log_reruns,
                emit=st.n_emit)

out = {}
os.environ["SFQED_WRITE_REPLAY"] = "0"
step(N)                       # the rest of the scratch
os.environ["SFQED_WRITE_REPLAY"] = "1"
out["none"] = [step(0), step(0)]
out["few"] = [step(100), step(100)]
hog = torch.empty(torch.cuda.mem_get_info()[0] - 900 * MIB, dtype=torch.uint8, device="cuda")
out["all"] = [step(N), step(N)]
out["few_after"] = [step(100)]
print("OUT " + json.dumps(out), flush=True)
"""


def test_log_takes_what_events_need():
    need_gpu()
    root = Path(__file__).resolve().parents[1]
    env = dict(os.environ, PYTHONPATH=str(root))
    r = subprocess.run([sys.executable, "-c", CHILD], env=env, cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    out = json.loads(next(ln for ln in r.stdout.splitlines() if ln.startswith("OUT "))[4:])
    print(out)
    mib = 1 << 20
    assert all(s["emit"] == 0 and s["reruns"] == 0 and s["taken"] <= 8 * mib for s in out["none"])
    first, second = out["few"]
    assert 10 < first["emit"] < 1000 and first["taken"] <= 40 * mib  # 100 neighbours are in a few waves
    assert second["replays"] == 1 and second["reruns"] == 0 and second["taken"] == 0
    # a need above half of what is left: written directly, step after step, and the small pool stays
    assert all(s["reruns"] == 1 and s["taken"] == 0 and s["emit"] > 100_000 for s in out["all"])
    assert out["few_after"][0]["replays"] == 1 and out["few_after"][0]["reruns"] == 0
