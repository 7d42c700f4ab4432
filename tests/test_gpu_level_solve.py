"""The leveling thresholds from the one-launch solve against the solve pass by
pass (which a block that may not wait for the others leaves to the host): the
same sums in the same order, so thresholds, iterations and survivors must be
equal bit for bit, at the edges of a slot (262144 particles), with the photon
filter and without, with empty species and targets that leave everything.  Above
35 slots the passes are launched one by one anyway; that size is checked against
the oracle's threshold."""
import numpy as np
import pytest

from oracle import resample as ors

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu
SLOT = 262144


def stores(sf, torch, n, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(9)

    def u(m):
        return torch.rand(m, dtype=torch.float64, device="cuda", generator=g)
    out = []
    for s in range(3):
        m = n[s]
        st = sf.Store.empty(max(m, 1), dtype, photon=s == 2)
        for c in (st.px, st.py, st.pz):
            c[:m] = (6 * u(m) - 3).to(dtype)
        st.w[:m] = torch.exp(4 * u(m) - 2).float()
        st.w[: m // 5] = 0.75
        st.tau[:m] = u(m)
        st.id[:m] = torch.arange(m, device="cuda") + (s << 40)
        if s == 2:
            st.alive[:m] = 1
        st.count = m
        out.append(st)
    return out


def resample(sf, torch, n, dtype, **cfg):
    main = stores(sf, torch, n, dtype)
    none = sf.Fields.from_array(np.zeros((1, 6)), dtype)
    st = sf.resample(main, [none] * 3, sf.resample_cfg(seed=7, step=3, **cfg))
    torch.cuda.synchronize()
    return main, st


@pytest.mark.parametrize("dtype_name", ["float32", "float64"])
@pytest.mark.parametrize("n, target, e_min", [
    ((1, 0, 0), (1, 1, 1), 0.0), ((3, 70, 1000), (1, 7, 40), 2.0), ((0, 5, 4099), (3, 9, 0), 2.0),
    ((SLOT - 1, SLOT, SLOT + 1), (60_000, 300_000, 1000), 0.0),
    ((2 * SLOT + 77, 129, 9 * SLOT + 5), (400_000, 128, 500_001), 2.0)])
def test_equals_the_passes(monkeypatch, dtype_name, n, target, e_min):
    torch, sf = need_gpu()
    dtype = getattr(torch, dtype_name)
    cfg = dict(target=target, photon_energy_min=e_min)
    monkeypatch.delenv("SFQED_LEVEL_WAIT_US", raising=False)
    ma, sa = resample(sf, torch, n, dtype, **cfg)
    monkeypatch.setenv("SFQED_LEVEL_WAIT_US", "0")
    mb, sb = resample(sf, torch, n, dtype, **cfg)
    assert list(sa.w_threshold) == list(sb.w_threshold) and list(sa.iterations) == list(sb.iterations)
    assert list(sa.count_after) == list(sb.count_after) and sa.filtered == sb.filtered
    for s in range(3):
        k = ma[s].count
        assert k == mb[s].count
        for name in ("px", "py", "pz", "w", "tau", "id"):
            assert torch.equal(getattr(ma[s], name)[:k], getattr(mb[s], name)[:k]), (s, name)


@pytest.mark.parametrize("n", [35 * SLOT, 35 * SLOT + 1])
def test_largest_one_launch_solve(n):
    torch, sf = need_gpu()
    w = stores(sf, torch, (n, 0, 0), torch.float32)[0].w[:n].cpu().numpy()
    main, st = resample(sf, torch, (n, 0, 0), torch.float32, target=(n // 3, 0, 0))
    ref = ors.leveling_threshold(w, n // 3)
    assert abs(st.w_threshold[0] - ref) <= 1e-11 * ref  # sums of 9e6 terms, in another order
    assert main[0].count == st.count_after[0] and abs(main[0].count - n // 3) < 5 * np.sqrt(n)
