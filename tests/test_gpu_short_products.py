"""Layers whose products are short (16 columns a workgroup, operands straight into registers, rows normalised on the way
in): against the oracle at the edges of its row tiles and of K, and one sequence's bits whatever shares its step."""
import numpy as np
import pytest
import torch

from oracle import ds_oracle as orc
from paper_2401_09670_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
TOL = 1e-2
CTX = 21

# Heads, head size, FFN.  Hidden sizes: the least K, waves with unequal shares of K, the longest rows that are normalised,
# longer ones, the longest K.  512 x 4096 is normalised in the FFN's product up to 32 rows and by a launch above: one row's
# bits are the same both ways.  (A layer's widths are multiples of 64: there is no last tile of fewer than 16 columns.)
LAYERS = [(4, 64, 1024), (6, 64, 256), (8, 64, 512), (8, 64, 4096), (10, 64, 1024), (8, 128, 4096)]


def _step(layer, batch, rows, context=CTX):
    """y, K and V rows of a step of `batch` sequences, the sequences `rows` of a larger one."""
    shape, ctx, lw, x, kc0, vc0, tables, nblk = layer
    kc, vc = kc0.clone(), vc0.clone()
    y = torch.full((batch + 1, shape.hidden), 7.0, dtype=torch.bfloat16, device="cuda")      # guard row
    ctx.ds_decode_step(lw, x[rows].contiguous(), gu.i32_dev([context] * batch), gu.i32_dev(tables[rows]), batch,
                       tables.shape[1], context + 1, kc, vc, nblk, y,
                       gu.workspace(ctx.ds_decode_workspace_bytes(batch, context + 1)))
    torch.cuda.synchronize()
    assert bool((y[batch] == 7.0).all()), "wrote past the last row"
    return y[:batch], kc, vc


@pytest.mark.parametrize("heads,head_dim,ffn", LAYERS)
def test_short_products_of_a_step(gpu, heads, head_dim, ffn):
    shape = synth.ModelShape(hidden=heads * head_dim, n_heads=heads, head_dim=head_dim, ffn=ffn)
    most = 64
    wbits = synth.make_layer_weights(shape, 91)
    lw, keep = gu.weights_to_dev(wbits)
    ctx = gu.make_ctx(shape)
    assert ctx.ds_layer_plan(1, shape.hidden, shape.qkv_width)["tile_cols"] == 16
    tables, nblk = synth.make_block_tables([CTX + 1] * most, 16, 3)
    kc0, vc0 = (gu.dev_normal_bits((nblk, shape.kv_heads, 16, head_dim), 1.0, i) for i in (1, 2))
    x = gu.dev_normal_bits((most, shape.hidden), 1.0, 5)
    layer = (shape, ctx, lw, x, kc0, vc0, tables, nblk)
    want = orc.layer_decode_cached(orc.weights_from_bits(wbits), gu.to_f64(x), [CTX] * most, tables, gu.to_f64(kc0),
                                   gu.to_f64(vc0), heads)
    full, kc, vc = _step(layer, most, list(range(most)))
    for batch in (1, 2, 4, 5, 8, 9, 12, 13, 15, 16, 17, 32, 33, 48, 49, 63):
        rows = [(7 * i + 1) % most for i in range(batch)]
        got, kb, vb = _step(layer, batch, rows)
        assert torch.equal(got, full[rows]), batch
        g, xin = gu.to_f64(got), gu.to_f64(x[rows])
        assert gu.rel_err_rows(g, want[rows]) < TOL and gu.update_ok(g, want[rows], xin), batch
        for i in (0, batch - 1):          # this step's K and V rows
            blk = int(tables[rows[i]][CTX // 16])
            assert torch.equal(kb[blk, :, CTX % 16], kc[blk, :, CTX % 16])
            assert torch.equal(vb[blk, :, CTX % 16], vc[blk, :, CTX % 16])


@pytest.mark.parametrize("heads,ffn,most", [(4, 1024, 64), (8, 2048, 32)])
def test_steps_at_longer_contexts_normalise_in_their_products(gpu, heads, ffn, most):
    """Where the attention would start its sequences in an order of its own, too: no LayerNorm launch, and a sequence's K
    and V rows are those of a smaller step."""
    context = 300
    shape = synth.ModelShape(hidden=heads * 64, n_heads=heads, head_dim=64, ffn=ffn)
    lw, keep = gu.dev_layer_weights(shape, 93)
    ctx = gu.make_ctx(shape)
    tables, nblk = synth.make_block_tables([context + 1] * most, 16, 3)
    kc0, vc0 = (gu.dev_normal_bits((nblk, heads, 16, 64), 1.0, i) for i in (1, 2))
    layer = (shape, ctx, lw, gu.dev_normal_bits((most, shape.hidden), 1.0, 5), kc0, vc0, tables, nblk)
    ctx.ds_profile_enable(True)
    _, kc, vc = _step(layer, most, list(range(most)), context)
    assert ctx.ds_profile_collect()["layernorm"][1] == 0
    ctx.ds_profile_enable(False)
    rows = [(7 * i + 1) % most for i in range(5)]
    _, kb, vb = _step(layer, 5, rows, context)
    for r in rows:
        blk = int(tables[r][context // 16])
        assert torch.equal(kb[blk, :, context % 16], kc[blk, :, context % 16])
        assert torch.equal(vb[blk, :, context % 16], vc[blk, :, context % 16])


@pytest.mark.parametrize("t", [1, 16, 17, 50, 64])
@pytest.mark.parametrize("heads,head_dim,ffn", LAYERS[:2])
def test_short_products_of_a_prompt(gpu, heads, head_dim, ffn, t):
    shape = synth.ModelShape(hidden=heads * head_dim, n_heads=heads, head_dim=head_dim, ffn=ffn)
    wbits = synth.make_layer_weights(shape, 92)
    lw, keep = gu.weights_to_dev(wbits)
    ctx, h = gu.make_ctx(shape), shape.hidden
    xbits = synth.make_activations(t, h, 92)
    y, k, v = (torch.full((t + 1, h), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(3))
    ctx.ds_prefill(lw, gu.to_dev(xbits), gu.i32_dev([0, t]), 1, t, t, y, k, v,
                   gu.workspace(ctx.ds_prefill_workspace_bytes(t)))
    torch.cuda.synchronize()
    x = orc.from_bf16_bits(xbits)
    yr, kr, vr = orc.layer_prefill(orc.weights_from_bits(wbits), x, [t], heads)
    assert all(bool((o[t] == 7.0).all()) for o in (y, k, v)), "wrote past the last row"
    assert gu.rel_err_rows(gu.to_f64(y[:t]), yr) < TOL and gu.update_ok(gu.to_f64(y[:t]), yr, x)
    for got, ref in ((k, kr), (v, vr)):
        assert gu.rel_err_rows(gu.to_f64(got[:t]), ref.reshape(t, h)) < TOL
