"""ds_layer_plan against the kernels that ds_decode_step launches, read off their names: family, tile, whether a reduce
pass follows (splits), whether the product is cut."""
import re

import pytest
import torch

from paper_2401_09670_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _kernels(call):
    call()
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    device = [e for e in prof.events() if e.device_type == torch.autograd.DeviceType.CUDA]
    return [e.name for e in sorted(device, key=lambda e: e.time_range.start)]


def _products_of(names):
    """[(streaming, tile rows or 0, columns, split?)] of the launches that multiply, in order."""
    out = []
    for name in names:
        arg = re.search(r"(gemm_dl|skinny_gemm|wring_gemm)_kernel<([^>]*)>", name)
        if arg:
            v = [a.strip() for a in arg.group(2).split(",")]
            if arg.group(1) == "gemm_dl":
                out.append([False, int(v[0]), int(v[1]), False])
            else:
                out.append([True, 0, 64 * int(v[1]) if arg.group(1) == "skinny_gemm" else 16 * int(v[0]), False])
        elif "skinny_reduce" in name:
            out[-1][3] = True
    return [tuple(p) for p in out]


def _step(shape, batch):
    ctx = gu.make_ctx(shape)
    lw, keep = gu.dev_layer_weights(shape, 7)
    h = shape.hidden
    lens = [3] * batch
    tables, nblk = synth.make_block_tables([4] * batch, 16, 5)
    kc, vc = (gu.dev_normal_bits((nblk, shape.kv_heads, 16, shape.head_dim), 1.0, i) for i in (1, 2))
    x, y = gu.dev_normal_bits((batch, h), 1.0, 3), torch.empty(batch, h, dtype=torch.bfloat16, device="cuda")
    lens, tab, ws = gu.i32_dev(lens), gu.i32_dev(tables), gu.workspace(ctx.ds_decode_workspace_bytes(batch, 4))
    names = _kernels(lambda: ctx.ds_decode_step(lw, x, lens, tab, batch, tables.shape[1], 4, kc, vc, nblk, y, ws))
    return ctx, names


@pytest.mark.parametrize("heads,head_dim,ffn,n_kv,batch", [
    (4, 64, 1024, 0, 2), (4, 64, 1024, 0, 8), (4, 64, 1024, 0, 64), (8, 128, 4096, 0, 33),    # small: unsplit in a layer
    (96, 128, 512, 0, 4), (96, 128, 512, 0, 64),                                              # a wide out-projection
    (40, 128, 5248, 0, 48),
    (56, 128, 512, 0, 970), (72, 128, 512, 8, 1810), (16, 128, 512, 0, 6000),                 # QKV is cut at a column
    (96, 128, 512, 0, 512),
])
def test_what_is_reported_is_what_runs(gpu, heads, head_dim, ffn, n_kv, batch):
    shape = synth.ModelShape(hidden=heads * head_dim, n_heads=heads, head_dim=head_dim, ffn=ffn, n_kv_heads=n_kv)
    ctx, names = _step(shape, batch)
    h, m = shape.hidden, shape.ffn
    ran = _products_of(names)
    for k, n in ((h, shape.qkv_width), (h, h), (h, m), (m, h)):
        p = ctx.ds_layer_plan(batch, k, n)
        assert ran.pop(0) == (p["streaming"], p["tile_rows"], p["tile_cols"], p["splits"] > 1), (k, n, p, names)
        if p["cut_cols"]:
            assert not ran.pop(0)[0]
    assert not ran
