"""The sum of the per-wave partial gradients (rows of a batch) over every split
of rows among the reducing threads: fewer rows than threads, exactly as many,
one row group more, and many.

Sums are compared with the same kernel's gradients over chunks of 64 samples
(two rows each) added in FP64.  Batch sizes are 64 times a power of two, so a
chunk's gradient (scaled by 1 / 64) and its share of the batch's (by 1 / n)
differ by an exact power of two through every rounding; what remains is the
rounding to FP32 of each chunk's sum and of the total, 2^-24 of each."""
import numpy as np
import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunks", [1, 2, 8, 16, 32, 256])
def test_rows_of_a_batch_add_up(chunks):
    torch, sf = need_gpu()
    n = 64 * chunks
    g = np.random.default_rng(3)
    net = sf.Mlp(g.normal(scale=0.3, size=sf.MLP_PARAMS).astype(np.float32))
    x = torch.tensor(np.stack([g.uniform(-1, 1, n), g.uniform(-2, 2, n)], 1).astype(np.float32), device="cuda")
    t = torch.tensor(g.normal(size=n).astype(np.float32), device="cuda")
    total, loss = (v.cpu().double() for v in net.grad(x, t))
    want, bound, sq = torch.zeros_like(total), torch.zeros_like(total), 0.0
    for c in range(chunks):
        part, lc = (v.cpu().double() for v in net.grad(x[64 * c:64 * c + 64].contiguous(), t[64 * c:64 * c + 64]
                                                       .contiguous()))
        want += part / chunks
        bound += part.abs() / chunks
        sq += float(lc) / chunks
    assert ((total - want).abs() <= 2.0 ** -23 * bound + 1e-30).all()
    assert abs(float(loss) - sq) <= 2.0 ** -23 * sq
