"""Which way a leveling solve went, and what it cost: one launch on an idle GPU;
a block that gives up (a wait of 0 or 1 us) leaves the rest to passes that are
queued together, two read-backs for the whole call; after a time-out the next
solves do not try again at once; and a solve of more passes than the launch makes
goes on where it stopped.  The results are the same bits each way."""
import numpy as np
import pytest

import test_gpu_level_solve as base
from gpu_util import need_gpu

pytestmark = pytest.mark.gpu
COLS = ("px", "py", "pz", "w", "tau", "id")


def same(torch, a, b):
    (ma, sa), (mb, sb) = a, b
    assert list(sa.w_threshold) == list(sb.w_threshold) and list(sa.iterations) == list(sb.iterations)
    assert list(sa.count_after) == list(sb.count_after) and sa.filtered == sb.filtered
    for s in range(3):
        for name in COLS:
            n = ma[s].count
            assert torch.equal(getattr(ma[s], name)[:n], getattr(mb[s], name)[:n]), (s, name)


def until_one_launch(call, limit=17):
    """Calls until a solve runs in one launch again (after a time-out, 16 of them do not)."""
    for k in range(limit):
        r = call()
        if r[1].one_launch:
            return k, r
        assert r[1].read_backs == 1
    raise AssertionError("no solve in one launch")


@pytest.mark.parametrize("dtype_name", ["float32", "float64"])
@pytest.mark.parametrize("n", [(3, 70, 1000), (base.SLOT + 77, 5000, 2 * base.SLOT + 5)])
def test_ways_and_waits(monkeypatch, dtype_name, n):
    torch, sf = need_gpu()
    dtype = getattr(torch, dtype_name)
    cfg = dict(target=tuple(max(1, m // 3) for m in n), photon_energy_min=2.0)

    def call():
        return base.resample(sf, torch, n, dtype, **cfg)
    monkeypatch.delenv("SFQED_LEVEL_WAIT_US", raising=False)
    _, one = until_one_launch(call)
    assert one[1].one_launch == 1 and one[1].read_backs == 1
    assert 2 <= max(one[1].iterations) <= 7  # fewer than the passes that are queued at most
    monkeypatch.setenv("SFQED_LEVEL_WAIT_US", "0")
    for _ in range(2):
        zero = call()
        assert zero[1].one_launch == 0 and zero[1].read_backs == 2
        same(torch, one, zero)
    monkeypatch.delenv("SFQED_LEVEL_WAIT_US")
    assert until_one_launch(call)[0] == 0  # a wait of 0 says nothing about the chip
    monkeypatch.setenv("SFQED_LEVEL_WAIT_US", "1")
    late = call()
    assert late[1].one_launch == 0 and late[1].read_backs == 2
    same(torch, one, late)
    monkeypatch.delenv("SFQED_LEVEL_WAIT_US")
    calls, again = until_one_launch(call)
    assert calls == 16
    same(torch, one, again)


def test_more_passes_than_the_launch_makes(monkeypatch):
    torch, sf = need_gpu()
    # a geometric series over 74 decades, one particle too many: the solve goes through it step by step
    w = np.float32(1e37) * np.float64(1.15) ** -np.arange(1215)
    w = w[w > 1e-37].astype(np.float32)
    n = w.size
    none = sf.Fields.from_array(np.zeros((1, 6)), torch.float32)

    def call():
        p = np.ones((n, 3))
        main = [sf.Store.from_arrays(p[:k], w[:k], np.ones(k), np.arange(k, dtype=np.uint64), dtype=torch.float32,
                                     photon=s == 2, capacity=max(k, 1)) for s, k in enumerate((n, 0, 0))]
        return main, sf.resample(main, [none] * 3, sf.resample_cfg(target=(n - 1, 0, 0), seed=1, step=2))
    monkeypatch.delenv("SFQED_LEVEL_WAIT_US", raising=False)
    call()  # queues as many passes as it may from here on
    for _ in range(17):
        a = call()
    monkeypatch.setenv("SFQED_LEVEL_WAIT_US", "0")
    b = call()
    assert a[1].iterations[0] > 40 and a[1].one_launch == 0
    # 32 passes in the launch, then 8 at a time; without it 9, then 8 at a time
    assert a[1].read_backs == 1 + (a[1].iterations[0] - 31 + 7) // 8
    assert b[1].read_backs == 2 + (b[1].iterations[0] - 8 + 7) // 8
    same(torch, a, b)


def test_filter_alone_is_one_pass():
    torch, sf = need_gpu()
    n = (300, 5000, 70_001)
    for _ in range(2):
        main, st = base.resample(sf, torch, n, torch.float32, photon_energy_min=2.0)
        assert st.one_launch == 0 and st.read_backs == 1
        assert list(st.count_after[:2]) == [300, 5000] and st.filtered == n[2] - main[2].count > 0
        main, st = base.resample(sf, torch, n, torch.float32, photon_energy_min=1e-6)
        assert st.read_backs == 1 and st.filtered == 0 and list(st.count_after) == list(n)
