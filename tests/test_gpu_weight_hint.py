"""Which launches load their weights with the non-temporal hint, read off the kernels that ran (the template's last
argument): those of at most eight row tiles over weights of 96 MB and more in a layer, of 256 MB and more in ds_linear."""
import re

import pytest
import torch

from paper_2401_09670_amd import binding, synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
TILE, PARTIAL, KV_SCATTER, HINT = slice(0, 2), 1, 2, 7


def _tile_kernels(call):
    """Template arguments of every tile GEMM that `call` launches."""
    call()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    found = []
    for e in prof.events():
        args = re.search(r"gemm_dl_kernel<([^>]*)>", e.name)
        if args:
            v = [a.strip() for a in args.group(1).split(",")]
            found.append([int(a) for a in v[:7]] + [v[7] == "true"])
    return found


def _linear(m, k, n):
    ctx = binding.Context(5120, 40, 128, 20480)
    x, w = gu.dev_normal_bits((m, k), 1.0, 1), gu.dev_normal_bits((n, k), 0.02, 2)
    y, ws = torch.empty(m, n, dtype=torch.bfloat16, device="cuda"), gu.workspace(ctx.ds_linear_workspace_bytes(m, k, n))
    return _tile_kernels(lambda: ctx.ds_linear(x, w, None, None, 0, m, k, n, y, ws))


@pytest.mark.parametrize("m,k,n,hint", [
    (33, 2112, 5120, False),       # 64x128 tiles (K no multiple of 128), 22 MB
    (33, 8256, 16384, True),       # ... 271 MB
    (129, 8192, 8192, False),      # 134 MB, split
    (300, 8192, 16376, True),      # 268 MB
    (300, 8192, 15360, False),     # 252 MB
    (2400, 8192, 16376, False),    # more than eight row tiles
])
def test_linear_takes_the_hint_beyond_the_last_level_cache(gpu, m, k, n, hint):
    kernels = _linear(m, k, n)
    assert kernels and all(a[HINT] == hint for a in kernels)


def _layer_kernels(heads, ffn, rows, decode, n_kv=0):
    h = heads * 128
    shape = synth.ModelShape(hidden=h, n_heads=heads, head_dim=128, ffn=ffn, n_kv_heads=n_kv)
    ctx = gu.make_ctx(shape)
    lw, keep = gu.dev_layer_weights(shape, 7)
    x, y = gu.dev_normal_bits((rows, h), 1.0, 3), torch.empty(rows, h, dtype=torch.bfloat16, device="cuda")
    if decode:
        tables, nblk = synth.make_block_tables([5] * rows, 16, 5)
        kc, vc = (gu.dev_normal_bits((nblk, shape.kv_heads, 16, 128), 1.0, i) for i in (1, 2))
        lens, tab, ws = gu.i32_dev([4] * rows), gu.i32_dev(tables), gu.workspace(ctx.ds_decode_workspace_bytes(rows, 5))
        return _tile_kernels(lambda: ctx.ds_decode_step(lw, x, lens, tab, rows, tables.shape[1], 5, kc, vc, nblk, y, ws))
    k, v = (torch.empty(rows, shape.kv_heads, 128, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    cu, ws = gu.i32_dev([0, rows]), gu.workspace(ctx.ds_prefill_workspace_bytes(rows))
    return _tile_kernels(lambda: ctx.ds_prefill(lw, x, cu, 1, rows, rows, y, k, v, ws))


@pytest.mark.parametrize("decode", [False, True])
@pytest.mark.parametrize("rows", [129, 200, 300, 520])
def test_small_layers_keep_their_weights(gpu, rows, decode):
    """2048 x 8192 (8 to 34 MB a product), K and V scattered by unsplit tiles in a decoding step."""
    kernels = _layer_kernels(16, 8192, rows, decode)
    assert kernels and not any(a[HINT] for a in kernels)


@pytest.mark.parametrize("rows,decode", [(140, False), (300, False), (140, True)])
def test_layers_of_large_weights_stream_them(gpu, rows, decode):
    """8192 x 8192 (three products of 134 and more MB, the FFN's two)."""
    kernels = _layer_kernels(64, 8192, rows, decode, n_kv=8)
    assert len(kernels) >= 4 and all(a[HINT] for a in kernels)
