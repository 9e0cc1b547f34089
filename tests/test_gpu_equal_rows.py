"""Rows that are equal have equal bits in every output, wherever they lie in a batch: the row tiles of a column add K in
one order, also where workgroups start at different places of K (rows a multiple of 4 KB apart)."""
import pytest
import torch

from paper_2401_09670_amd import binding, synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,n", [(8192, 16392), (12288, 36872)])      # more than 256 MB of weights, a ragged last column tile
@pytest.mark.parametrize("m", [290, 700, 1500])
def test_linear_of_equal_rows(gpu, m, k, n):
    ctx = binding.Context(5120, 40, 128, 20480)
    x = gu.dev_normal_bits((1, k), 1.0, m).repeat(m, 1)
    w = gu.dev_normal_bits((n, k), 0.02, 7)
    y = torch.empty(m, n, dtype=torch.bfloat16, device="cuda")
    ctx.ds_linear(x, w, None, None, 0, m, k, n, y, gu.workspace(ctx.ds_linear_workspace_bytes(m, k, n)))
    torch.cuda.synchronize()
    assert torch.equal(y, y[:1].expand(m, n))


@pytest.mark.parametrize("heads,n_kv,prompts,length", [
    (64, 8, 4, 75), (64, 8, 3, 200), (64, 8, 5, 257),     # 8192 features in and 32768
    (48, 0, 7, 220),                                       # 6144 and 24576
])
def test_prefill_of_equal_prompts(gpu, heads, n_kv, prompts, length):
    h = heads * 128
    shape = synth.ModelShape(hidden=h, n_heads=heads, head_dim=128, ffn=4 * h, n_kv_heads=n_kv)
    ctx = gu.make_ctx(shape)
    lw, keep = gu.dev_layer_weights(shape, 31)
    t = prompts * length
    x = gu.dev_normal_bits((length, h), 1.0, 32).repeat(prompts, 1)
    y = torch.empty_like(x)
    k, v = (torch.empty(t, shape.kv_heads, 128, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    ctx.ds_prefill(lw, x, gu.i32_dev([length * i for i in range(prompts + 1)]), prompts, t, length, y, k, v,
                   gu.workspace(ctx.ds_prefill_workspace_bytes(t)))
    torch.cuda.synchronize()
    for out in (k, v, y):
        per = out.view(prompts, length, -1)
        assert torch.equal(per, per[:1].expand_as(per))
