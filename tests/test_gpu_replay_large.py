"""The replay of large launches (more than 256 leptons per SIMD) against the
direct write kernel, over the forms it is compiled for: by lanes in FP32 and in
FP64 with push or positions, by events in FP64 without either, sources in the
ensemble and in records, with and without the counters of launches above 512
particles per wave.  Records, positions, final states and counts must be the
same bits."""
import numpy as np
import pytest

import synth

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu
BY_LANES = 256 * 4 * 256  # leptons of a launch on 256 CUs, above which it is replayed by lanes


@pytest.mark.parametrize("push", [False, True])
@pytest.mark.parametrize("positions", [False, True])
@pytest.mark.parametrize("dtype_name", ["float32", "float64"])
@pytest.mark.parametrize("n", [132_001, 1_060_003])  # of each species
def test_equals_direct_writes(monkeypatch, dtype_name, push, positions, n):
    torch, sf = need_gpu()
    dtype = getattr(torch, dtype_name)
    photons = max(n, 300_000)
    wl = synth.crossed_field(10_000_000, indices=[np.arange(n), np.arange(n) + 5, np.arange(photons)])
    wl.species[2].tau[:] *= 1e-6  # nearly every photon makes a pair at once: the next round's leptons are records
    rng = np.random.default_rng(4)
    x0 = [rng.normal(0.0, 1e3, (sp.n, 3)) for sp in wl.species]
    fields = [sf.Fields.from_array(sp.fields, dtype) for sp in wl.species]
    tabs = sf.Tables()
    cfg = sf.step_cfg(push=push, gamma_min=2.0, nev=not push)
    cap = [photons + n // 4, photons + n // 4, 12 * n + 8 * photons]

    def run(replay):
        monkeypatch.setenv("SFQED_WRITE_REPLAY", replay)
        main = [sf.Store.from_arrays(sp.p, sp.w, sp.tau, sp.id, dtype=dtype, photon=s == 2,
                                     x=x0[s] if positions else None) for s, sp in enumerate(wl.species)]
        app = [sf.AppendBuffer(c, dtype, positions=positions) for c in cap]
        for a in app:
            a.data.zero_()
        _, st = sf.step(tabs, main, fields, app, wl.dt * 0.02, 5, 1, cfg)
        return main, app, st

    ma, aa, sa = run("0")
    run("1")  # grows the log's pool if it has to
    mb, ab, sb = run("1")
    assert sb.log_replays > 0 and sb.log_reruns == 0
    assert 2 * n > BY_LANES and 2 * sb.n_pair > BY_LANES, sb.n_pair
    assert n // 2 < sa.n_emit == sb.n_emit and sa.n_rounds == sb.n_rounds >= 2
    for s in range(3):
        for name in ("px", "py", "pz", "tau", "nev") + (("x", "y", "z") if positions else ()):
            assert torch.equal(getattr(ma[s], name), getattr(mb[s], name)), (s, name)
        assert aa[s].count == ab[s].count
        assert torch.equal(aa[s].data, ab[s].data), s
        if positions:
            assert torch.equal(aa[s].pos[:aa[s].count], ab[s].pos[:ab[s].count]), s
