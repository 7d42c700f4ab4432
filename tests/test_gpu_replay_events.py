"""The write pass that replays a small launch's events in parallel against the
direct write kernel, over the forms it is compiled for: FP32 and FP64, push and
positions on and off, sources in the ensemble and in records, one event per
particle up to chains far longer than a tile of trips, event counts written
or not.  Records, positions, final states and counts must be the same bits."""
import numpy as np
import pytest

import synth

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype_name", ["float32", "float64"])
@pytest.mark.parametrize("push", [False, True])
@pytest.mark.parametrize("positions", [False, True])
@pytest.mark.parametrize("n, dt", [(7, 1.0), (800, 1.0), (20_000, 0.05)])
def test_equals_direct_writes(monkeypatch, dtype_name, push, positions, n, dt):
    torch, sf = need_gpu()
    dtype = getattr(torch, dtype_name)
    wl = synth.crossed_field(10_000_000, indices=[np.arange(n), np.arange(n) + 5, np.arange(n // 4 + 1)])
    rng = np.random.default_rng(3)
    tabs = sf.Tables()
    cfg = sf.step_cfg(push=push, gamma_min=2.0, nev=not push)
    cap = [8 * n + 4000, 8 * n + 4000, 150 * n + 40_000]
    x0 = [rng.normal(0.0, 1e3, (sp.n, 3)) for sp in wl.species]

    def run(replay):
        monkeypatch.setenv("SFQED_WRITE_REPLAY", replay)
        main, fields, app = [], [], []
        for s, sp in enumerate(wl.species):
            main.append(sf.Store.from_arrays(sp.p, sp.w, sp.tau, sp.id, dtype=dtype, photon=s == 2,
                                             x=x0[s] if positions else None))
            fields.append(sf.Fields.from_array(sp.fields, dtype))
            app.append(sf.AppendBuffer(cap[s], dtype, positions=positions))
        _, st = sf.step(tabs, main, fields, app, wl.dt * dt * (0.02 if push else 1.0), 5, 1, cfg)
        return main, app, st

    ma, aa, sa = run("0")
    run("1")  # grows the log's pool if it has to
    mb, ab, sb = run("1")
    assert sb.log_replays > 0 and sb.log_reruns == 0
    assert sa.n_emit == sb.n_emit > 0 and sa.n_rounds == sb.n_rounds
    for s in range(3):
        A, B = ma[s].host(), mb[s].host()
        for name in A:
            assert np.array_equal(A[name], B[name]), (s, name)
        assert aa[s].count == ab[s].count
        assert torch.equal(aa[s].data, ab[s].data), s
        if positions:
            assert torch.equal(aa[s].pos, ab[s].pos), s
