"""Decoding batches whose workgroups queue start their longest sequences first: every sequence is still attended once,
over its own pages, whatever its place in the order."""
import numpy as np
import pytest
import torch

from paper_2401_09670_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,n_kv,batch", [
    (8, 0, 64),      # 512 workgroups: none queues, no order
    (8, 0, 65),      # 520
    (8, 0, 300),     # more sequences than the sorting workgroup has threads
    (8, 0, 512),     # as many as it sorts
    (8, 0, 513),     # one more: no order
    (16, 4, 140),    # grouped queries
])
@pytest.mark.parametrize("lengths", ["ragged", "equal"])
def test_batched_sequences_equal_single_ones(gpu, heads, n_kv, batch, lengths):
    h = heads * 128
    shape = synth.ModelShape(hidden=h, n_heads=heads, head_dim=128, ffn=256, n_kv_heads=n_kv)
    ctx = gu.make_ctx(shape)
    lw, keep = gu.dev_layer_weights(shape, 90 + batch)
    rng = np.random.Generator(np.random.Philox(key=[batch, heads]))
    lens = [int(v) for v in rng.integers(0, 40, batch)] if lengths == "ragged" else [33] * batch
    if lengths == "ragged":
        lens[batch // 2], lens[-1], lens[0] = 300, 299, 0
    tables, nblk = synth.make_block_tables([l + 1 for l in lens], 16, 7)
    kc0 = gu.dev_normal_bits((nblk, shape.kv_heads, 16, 128), 1.0, 1)
    vc0 = gu.dev_normal_bits((nblk, shape.kv_heads, 16, 128), 1.0, 2)
    x = gu.dev_normal_bits((batch, h), 1.0, 3)

    def step(rows):
        kc, vc = kc0.clone(), vc0.clone()
        y = torch.empty(len(rows), h, dtype=torch.bfloat16, device="cuda")
        sub = [lens[r] for r in rows]
        ws = gu.workspace(ctx.ds_decode_workspace_bytes(len(rows), max(lens) + 1))
        ctx.ds_decode_step(lw, x[rows].contiguous(), gu.i32_dev(sub), gu.i32_dev(tables[rows]), len(rows),
                           tables.shape[1], max(lens) + 1, kc, vc, nblk, y, ws)
        torch.cuda.synchronize()
        return gu.to_f64(y)

    batched = step(list(range(batch)))
    xin = gu.to_f64(x)
    for r in sorted({0, 1, batch // 2, batch - 2, batch - 1, *(int(v) for v in rng.integers(0, batch, 8))}):
        alone = step([r])
        assert gu.rel_err(batched[r:r + 1], alone) < 1e-2 and gu.update_ok(batched[r:r + 1], alone, xin[r:r + 1]), r
