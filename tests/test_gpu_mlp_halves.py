"""A wave of the surrogate's inference takes 32 samples of a small call and 64 of
a large one.  A sample's result depends on its inputs alone, so a large call
must equal the same samples in small calls bit for bit; the sizes end inside
the first and the second half of a wave's samples, around the size from which
waves take 64."""
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("past", [0, 1, 31, 33, 64, 100_003])
def test_large_calls_equal_small_ones(past):
    torch, sf = need_gpu()
    n = 32 * 8 * 4 * torch.cuda.get_device_properties(0).multi_processor_count + past
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    net, tabs = sf.Mlp(sf.load_surrogate()), sf.Tables()
    x = 4 * torch.rand(n, 2, device="cuda", generator=g) - 2
    chi = torch.exp(6 * torch.rand(n, device="cuda", generator=g) - 3)
    chi[::97] = 1e-3  # outside the trained range: the tables
    k = torch.randint(-2 ** 31, 2 ** 31, (n,), dtype=torch.int32, device="cuda", generator=g)
    y, d = net.forward(x), net.sample(tabs, chi, k)
    step = 100_000
    for a in range(0, n, step):
        assert torch.equal(y[a:a + step], net.forward(x[a:a + step].contiguous()))
        assert torch.equal(d[a:a + step], net.sample(tabs, chi[a:a + step].contiguous(), k[a:a + step].contiguous()))
