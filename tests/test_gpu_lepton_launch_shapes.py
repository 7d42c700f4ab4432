"""How a lepton launch deals its particles out to waves must not show in the
results: a particle's events depend on its own state, id and draws alone.  One
launch large enough for the counters (more than 512 particles per wave) is the
reference; smaller launches of its first particles, at the edges of the pieces
and of one, two and four waves per SIMD, must give the same final states, event
counts and records, bit for bit."""
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu
N = 2_200_003  # electrons of the reference launch; 2^21 is where the counters begin on 256 CUs


def ensemble(sf, torch, dtype, n, positrons, p, f, tau):
    main, fields, app = [], [], []
    for s in range(3):
        k = (n, positrons, 0)[s]
        st = sf.Store.empty(max(k, 1), dtype, photon=s == 2)
        st.px[:k], st.py[:k], st.pz[:k] = (c[:k] for c in p)
        st.w[:k] = 1.0
        st.tau[:k] = tau[:k]
        st.id[:k] = torch.arange(k, device="cuda") + (s << 32)
        st.count = k
        main.append(st)
        fields.append(sf.Fields(*[c[:max(k, 1)].contiguous() for c in f], stride=1))
        app.append(sf.AppendBuffer(3 * (n + positrons) + 4096 if s == 2 else 1, dtype))
    return main, fields, app


@pytest.mark.parametrize("dtype_name", ["float32", "float64"])
def test_results_do_not_depend_on_the_launch(dtype_name):
    torch, sf = need_gpu()
    dtype = getattr(torch, dtype_name)
    g = torch.Generator(device="cuda")
    g.manual_seed(11)

    def u(*shape):
        return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)
    p = [(100.0 * torch.exp(4.6 * u(N)) * d).to(dtype) for d in (0.6, -0.48, 0.64)]
    f = [torch.zeros(N, dtype=dtype, device="cuda") for _ in range(3)]
    f += [(1e-3 * (u(N) - 0.5)).to(dtype) for _ in range(3)]
    tau = -torch.log(u(N).clamp_min(1e-12))
    tabs = sf.Tables()
    cfg = sf.step_cfg(pair=False, push=False)

    def run(n, positrons):
        main, fields, app = ensemble(sf, torch, dtype, n, positrons, p, f, tau)
        rc, st = sf.step(tabs, main, fields, app, 2.0e5, 5, 1, cfg)
        torch.cuda.synchronize()
        return main, app[2], st

    ref, ref_app, st = run(N, 0)
    assert 0.2 * N < st.n_emit < 2 * N  # events to get wrong
    rec = ref_app.rec_dtype.itemsize
    root = ref_app.data[: st.n_emit * rec].view(torch.int32).reshape(st.n_emit, rec // 4)[:, rec // 4 - 3]
    for n in (1, 63, 64, 65, 255, 257, 1024, 65_537, 262_143, 262_145, 300_001, 1_048_577, 2_097_153):
        main, app, s = run(n, 0)
        for name in ("px", "py", "pz", "tau", "nev"):
            assert torch.equal(getattr(main[0], name)[:n], getattr(ref[0], name)[:n]), (n, name)
        kids = int((root < n).sum())
        assert s.n_emit == kids
        assert torch.equal(app.data[: kids * rec], ref_app.data[: kids * rec]), n
    # two source ranges: the boundary between species falls inside a piece
    main, _, _ = run(100_001, 70_003)
    one, _, _ = run(100_001, 0)
    for name in ("px", "py", "pz", "tau", "nev"):
        assert torch.equal(getattr(main[0], name), getattr(one[0], name)), name
    two, _, _ = run(0, 70_003)
    for name in ("px", "py", "pz", "tau", "nev"):
        assert torch.equal(getattr(main[1], name), getattr(two[1], name)), name
