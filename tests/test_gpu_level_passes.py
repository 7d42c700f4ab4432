"""Leveling solves above the size of the one-launch solve (35 slots of 262,144
particles): passes queued for the three species together, with the photon
filter's mask from the first of them, solves that need different numbers of
passes, and, after solves that needed one, too few passes queued ahead.
Checked against the oracle like the other resampling tests."""
import numpy as np
import pytest

import test_gpu_resample as base
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu
N = (300_001, 70_001, 8_912_900)  # 2 + 1 + 35 slots


def read_backs(iterations, queued):
    """of a call that queues `queued` passes after the first, and as many again until the last solve is done"""
    return 1 + -(-max(0, max(iterations) - queued) // queued)


@pytest.mark.parametrize("dtype_name", ["float32", "float64"])
def test_queued_passes(dtype_name):
    torch, sf = need_gpu()
    dtype = getattr(torch, dtype_name)
    data = base.ensemble(N, 21)
    # equal weights: w_0 = total / target is already the root, one pass confirms it
    flat = [(p, np.full_like(w, 0.75), tau, ids, x) for (p, w, tau, ids, x) in data]
    _, st = base.run(torch, sf, flat, dtype, dict(target=tuple(n // 4 for n in N), seed=3, step=1))
    assert list(st.iterations) == [1, 1, 1] and st.one_launch == 0 and st.read_backs <= 2
    kw = dict(photon_energy_min=2.0, target=(299_990, 10, 2_000_000), seed=7, step=3)
    main, few = base.run(torch, sf, data, dtype, kw)
    assert len(set(few.iterations)) > 1 and max(few.iterations) > 2
    # as many passes as the last solves took, and one: too few
    assert few.one_launch == 0 and few.read_backs == read_backs(few.iterations, 2) > 1
    for s in range(3):
        base.check_species(sf, main[s], data[s], s, few, kw, np.dtype(dtype_name).type)
    again, st = base.run(torch, sf, data, dtype, kw)
    assert st.one_launch == 0 and st.read_backs == read_backs(st.iterations, min(8, max(st.iterations) + 1))
    assert list(st.iterations) == list(few.iterations) and list(st.w_threshold) == list(few.w_threshold)
    for s in range(3):
        a, b = main[s].host(), again[s].host()
        assert all(np.array_equal(a[k], b[k]) for k in a)
