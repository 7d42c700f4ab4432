"""Resampling of the three species in shared launches, at the sizes where the
leveling pass (64 photons to a mask word, 8 particles in flight per thread, a
grid of 262,144 threads) and the compaction (tiles of 2048) change course, and
with species that are empty, untouched or solved in different numbers of
passes.  Checked against the oracle like the other resampling tests."""
import numpy as np
import pytest

import test_gpu_resample as base
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype_name", ["float32", "float64"])
@pytest.mark.parametrize("n, target, e_min", [
    ((1, 0, 1), (0, 0, 0), 2.0),
    ((63, 64, 65), (20, 64, 21), 2.0),
    ((0, 2047, 2049), (0, 1000, 0), 3.0),
    ((2048, 1, 4097), (2047, 0, 4096), 0.0),
    ((5000, 300, 262_145), (10, 299, 100_000), 2.0),
    ((70_001, 70_001, 2_097_217), (69_999, 1, 700_001), 2.0),
])
def test_sizes(dtype_name, n, target, e_min):
    torch, sf = need_gpu()
    data = base.ensemble(n, 17 + n[2])
    kw = dict(photon_energy_min=e_min, target=target, seed=9, step=4)
    for _ in range(2):  # the second call queues as many passes as the first one's solves took
        main, st = base.run(torch, sf, data, getattr(torch, dtype_name), kw)
        for s in range(3):
            base.check_species(sf, main[s], data[s], s, st, kw, np.dtype(dtype_name).type)
            assert list(st.count_before) == list(n)
