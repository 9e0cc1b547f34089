"""ds_linear on both sides of the size from which its weights are loaded past the caches, and of the row count up to
which they are, against a float32 product."""
import pytest
import torch

from paper_2401_09670_amd import binding
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
K = 8192


@pytest.mark.parametrize("n", [15616, 15632])     # 255.9 and 256.1 MB of weights
@pytest.mark.parametrize("m", [129, 257, 2048, 2049])
def test_linear_beside_the_streamed_size(gpu, m, n):
    torch.manual_seed(m + n)
    ctx = binding.Context(5120, 40, 128, 20480)
    x = torch.empty((m, K), device="cuda").normal_().to(torch.bfloat16)
    w = torch.empty((n, K), device="cuda").normal_(0, 0.02).to(torch.bfloat16)
    y = torch.full((m + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")
    ctx.ds_linear(x, w, None, None, 0, m, K, n, y, gu.workspace(ctx.ds_linear_workspace_bytes(m, K, n)))
    torch.cuda.synchronize()
    assert bool((y[m] == 7.0).all()), "wrote past the last row"
    xf, wf = x.float(), w.float()
    ref = xf @ wf.t()
    # one rounding to bf16 (2^-8 of the value), and both sums' K additions in float32 (2^-24 each of the terms' size)
    bound = 2.0 ** -8 * ref.abs() + 2 * K * 2.0 ** -24 * (xf.abs() @ wf.abs().t())
    assert bool(((y[:m].float() - ref).abs() <= bound).all())
