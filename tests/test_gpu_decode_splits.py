"""Decode attention on few sequences: splits whose partial states reach into scratch that is dead while the attention runs,
and the least number of splits where there is no more room."""
import re

import pytest
import torch

from oracle import ds_oracle as orc
from paper_2401_09670_amd import binding, synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
TOL = 1e-2
GUARD = 1 << 16

# heads, key/value heads, head size, FFN, sequences, longest context.  More splits than the least: 4 instead of 3, 6
# instead of 4, 3 instead of 2, 20 instead of 13; with an FFN of 64 for some of them, as far as the room goes.
STEPS = [(8, 8, 128, 4096, 24, 700), (16, 2, 128, 8192, 66, 1500), (4, 4, 64, 1024, 64, 300), (16, 16, 64, 64, 8, 700),
         (10, 10, 128, 64, 4, 5200)]


def _problem(heads, n_kv, head_dim, ffn, batch, longest):
    shape = synth.ModelShape(hidden=heads * head_dim, n_heads=heads, head_dim=head_dim, ffn=ffn, n_kv_heads=n_kv)
    lens = [longest - 1 if i % 7 == 3 else (i * 37) % longest for i in range(batch)]
    tables, nblk = synth.make_block_tables([n + 1 for n in lens], 16, 3)
    kc, vc = (gu.dev_normal_bits((nblk, n_kv, 16, head_dim), 1.0, i) for i in (1, 2))
    return shape, gu.make_ctx(shape), lens, tables, nblk, kc, vc


def _least_workspace(ctx, q, lens, tables, longest, kc, vc, nblk):
    """Bytes below which ds_decode_attention refuses the call."""
    with pytest.raises(binding.DsError) as refused:
        ctx.ds_decode_attention(q, gu.i32_dev(lens), gu.i32_dev(tables), len(lens), tables.shape[1], longest, kc, vc,
                                nblk, torch.empty_like(q), gu.workspace(256)[:256])
    return int(re.search(r"workspace 256 < (\d+)", str(refused.value)).group(1))


@pytest.mark.parametrize("heads,n_kv,head_dim,ffn,batch,longest", STEPS)
def test_a_step_stays_within_the_workspace_it_asks_for(gpu, heads, n_kv, head_dim, ffn, batch, longest):
    """The oracle's values and the static step's bits, also from a larger workspace, and nothing written behind it."""
    shape, ctx, lens, tables, nblk, kc0, vc0 = _problem(heads, n_kv, head_dim, ffn, batch, longest)
    wbits = synth.make_layer_weights(shape, 17)
    lw, keep = gu.weights_to_dev(wbits)
    x = gu.dev_normal_bits((batch, shape.hidden), 1.0, 5)
    args = (gu.i32_dev(lens), gu.i32_dev(tables), batch, tables.shape[1], longest)

    def step(size):
        kc, vc, y = kc0.clone(), vc0.clone(), torch.empty_like(x)
        if size is None:
            ctx.ds_decode_step_static(lw, x, *args, kc, vc, nblk, y)
        else:
            ws = torch.full((size + GUARD,), 0xff, dtype=torch.uint8, device="cuda")
            ctx.ds_decode_step(lw, x, *args, kc, vc, nblk, y, ws[:size])
            assert bool((ws[size:] == 0xff).all()), "wrote past the workspace"
        torch.cuda.synchronize()
        return y, kc, vc

    asked = ctx.ds_decode_workspace_bytes(batch, longest)
    got = step(asked)
    for other in (step(None), step(4 * asked)):
        assert all(torch.equal(a, b) for a, b in zip(got, other))
    rows = [0, 3, batch - 1]                       # sequences are independent of each other
    xin = gu.to_f64(x)[rows]
    want = orc.layer_decode_cached(orc.weights_from_bits(wbits), xin, [lens[r] for r in rows], tables[rows],
                                   gu.to_f64(kc0), gu.to_f64(vc0), heads)
    y = gu.to_f64(got[0])[rows]
    assert gu.rel_err_rows(y, want) < TOL and gu.update_ok(y, want, xin)


@pytest.mark.parametrize("heads,n_kv,head_dim,ffn,batch,longest", STEPS)
def test_attention_with_more_and_with_the_least_workspace(gpu, heads, n_kv, head_dim, ffn, batch, longest):
    shape, ctx, lens, tables, nblk, kc, vc = _problem(heads, n_kv, head_dim, ffn, batch, longest)
    q = gu.dev_normal_bits((batch, shape.hidden), 1.0, 5)

    def attend(size):
        o = torch.empty_like(q)
        ws = torch.full((size + GUARD,), 0xff, dtype=torch.uint8, device="cuda")
        ctx.ds_decode_attention(q, gu.i32_dev(lens), gu.i32_dev(tables), batch, tables.shape[1], longest, kc, vc, nblk,
                                o, ws[:size])
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0xff).all()), "wrote past the workspace"
        return o

    least = _least_workspace(ctx, q, lens, tables, longest, kc, vc, nblk)
    asked = ctx.ds_decode_workspace_bytes(batch, longest)
    assert least <= asked
    full = attend(asked)
    assert torch.equal(full, attend(4 * asked))
    kd, vd = gu.to_f64(kc), gu.to_f64(vc)
    for out in (full, attend(least)):
        got = gu.to_f64(out).reshape(batch, heads, head_dim)
        for i in (1, 3, batch - 1):
            k, v = (orc.kv_gather(c, tables[i], lens[i]) for c in (kd, vd))
            want = orc.attention_rows(gu.to_f64(q[i:i + 1]).reshape(1, heads, head_dim), [lens[i] - 1], k, v)[0]
            assert gu.rel_err(got[i], want) < TOL, i


# Heads, key/value heads, sequences, longest context, whether more splits than the least are taken: on both sides of 1024
# workgroups (3 splits of 341 and 342 pairs and more), of 128 grouped pairs, of 8 heads that share a key, of 1280 tokens.
@pytest.mark.parametrize("heads,n_kv,batch,longest,more", [
    (64, 8, 42, 700, True), (64, 8, 43, 700, False), (64, 8, 47, 2048, False), (40, 40, 8, 700, True),
    (40, 40, 9, 700, False), (31, 31, 11, 700, True), (18, 18, 19, 700, False), (64, 8, 16, 700, True),
    (64, 8, 15, 700, False), (32, 2, 100, 1280, False), (32, 2, 100, 1281, True), (16, 2, 100, 700, True),
])
def test_where_more_splits_than_the_least_are_taken(gpu, heads, n_kv, batch, longest, more):
    """Other splits, other sums: the bits of a call with the least workspace tell."""
    _, _, lens, tables, nblk, kc, vc = _problem(heads, n_kv, 128, 1024, batch, longest)
    ctx = binding.Context(heads * 128, heads, 128, 4 * heads * 128, n_kv_heads=n_kv)
    q = gu.dev_normal_bits((batch, heads * 128), 1.0, 5)
    asked = ctx.ds_decode_workspace_bytes(batch, longest)
    outs = []
    for size in (_least_workspace(ctx, q, lens, tables, longest, kc, vc, nblk), asked):
        o = torch.empty_like(q)
        ctx.ds_decode_attention(q, gu.i32_dev(lens), gu.i32_dev(tables), batch, tables.shape[1], longest, kc, vc, nblk,
                                o, gu.workspace(size)[:size])
        outs.append(o)
    assert torch.equal(*outs) != more
