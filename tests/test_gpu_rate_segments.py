"""FP64 steps read the rate coefficients from the block's copy when the table has
at most 64 segments, from memory otherwise.  Tables from chi = 1.3e-9 (64
segments), 1.2e-9 (65) and 1e-13 (83) must give the events of the default one
(56): momenta and ids exactly (without a push they follow from the draws alone),
birth times and depths up to the difference of the tables' rates, 1e-12
relative over the events of a lepton (some hundred; a depth of as many units is
used up)."""
import numpy as np
import pytest

import synth

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chi_min", [1.3e-9, 1.2e-9, 1e-13])
def test_segments_past_the_copy(chi_min):
    torch, sf = need_gpu()
    n = 5000
    wl = synth.crossed_field(10_000_000, indices=[np.arange(n), np.arange(n), np.arange(1)])
    out = []
    for kw in ({}, dict(rate_chi_min=chi_min)):
        tabs = sf.Tables(sf.default_table_cfg(**kw))
        main, fields, app = [], [], []
        for s, sp in enumerate(wl.species):
            main.append(sf.Store.from_arrays(sp.p, sp.w, sp.tau, sp.id, dtype=torch.float64, photon=s == 2))
            fields.append(sf.Fields.from_array(sp.fields, torch.float64))
            app.append(sf.AppendBuffer(150 * n + 40_000 if s == 2 else 1, torch.float64))
        _, st = sf.step(tabs, main, fields, app, wl.dt, 5, 1, sf.step_cfg(pair=False, push=False))
        torch.cuda.synchronize()
        out.append((st.n_emit, [main[0].host(), main[1].host(), app[2].host()]))
    (na, ha), (nb, hb) = out
    assert na == nb > n
    for a, b in zip(ha, hb):
        assert np.array_equal(a["id"], b["id"]) and np.array_equal(a["p"], b["p"])
        assert np.abs(a["tau"] - b["tau"]).max() <= 1e-7
    assert np.abs(ha[2]["t_birth"] - hb[2]["t_birth"]).max() <= 1e-10 * wl.dt
