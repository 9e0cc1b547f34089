"""The products of a layer from 65 rows on, on every tile that their plans take: one OPT-13B layer over batches whose
rows end inside, at and just past a tile, against the oracle; the K/V scatter of unsplit QKV tiles; and the smallest
workspace a call is accepted with."""
import numpy as np
import pytest
import torch

from oracle import ds_oracle as orc
from paper_2401_09670_amd import binding, synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
TOL = 1e-2
H, M_FFN = 5120, 20480
PRODUCTS = ((H, 3 * H), (H, H), (H, M_FFN), (M_FFN, H))


def _layer(shape, seed):
    wbits = synth.make_layer_weights(shape, seed)
    lw, keep = gu.weights_to_dev(wbits)
    return dict(shape=shape, seed=seed, lw=lw, keep=keep, ctx=gu.make_ctx(shape), w64=orc.weights_from_bits(wbits))


@pytest.fixture(scope="module")
def layer(gpu):
    return _layer(synth.OPT_13B, 4711)


def _plan(ctx, rows, products=PRODUCTS):
    out = []
    for k, n in products:
        p = ctx.ds_layer_plan(rows, k, n)
        out.append("stream" if p["streaming"] else f"{p['tile_rows']}x{p['tile_cols']}/{p['splits']}")
    return out


def _prefill(layer, t, ws):
    h = layer["shape"].hidden
    xbits = synth.make_activations(t, h, layer["seed"], stream=t)
    y, k, v = (torch.full((t + 1, h), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(3))   # guard row
    layer["ctx"].ds_prefill(layer["lw"], gu.to_dev(xbits), gu.i32_dev([0, t]), 1, t, t, y, k, v, ws)
    torch.cuda.synchronize()
    return orc.from_bf16_bits(xbits), y, k, v


def _check(layer, x, y, k, v):
    t, h = x.shape
    rng = np.random.Generator(np.random.Philox(key=[t, 3]))
    rows = sorted({0, 1, 63, 64, t // 2, t - 2, t - 1, *(int(r) for r in rng.integers(0, t, 9))})
    yr, kr, vr = orc.layer_prefill_rows(layer["w64"], x, rows, layer["shape"].n_heads, layer["shape"].ln_eps)
    for out in (y, k, v):
        assert bool((out[t] == 7.0).all()), "wrote past the last row"
    yg = gu.to_f64(y[:t])[rows]
    assert gu.rel_err(yg, yr) < TOL and gu.rel_err_rows(yg, yr) < TOL and gu.update_ok(yg, yr, x[rows])
    for got, ref in ((k, kr), (v, vr)):
        assert gu.rel_err_rows(gu.to_f64(got[:t]), ref.reshape(t, h)) < TOL


@pytest.mark.parametrize("t,plan", [
    (70, ["96x192/3", "64x128/3", "stream", "96x192/9"]),
    (100, ["128x128/2", "64x128/3", "stream", "128x128/6"]),
    (160, ["160x192/3", "128x128/3", "160x192/2", "160x192/9"]),      # rows end with the tile
    (161, ["192x192/3", "128x128/3", "192x192/2", "192x192/9"]),      # one row more
    (193, ["224x192/3", "128x128/3", "224x192/2", "224x192/9"]),
    (230, ["128x128/1", "128x128/3", "256x160/2", "256x160/8"]),      # eight splits: they turn
    (287, ["288x192/3", "160x192/4", "288x192/2", "288x192/9"]),
    (289, ["320x192/3", "160x192/4", "160x192/1", "320x192/9"]),
    (383, ["192x128/1", "192x128/3", "192x192/1", "384x160/8"]),
    (520, ["192x192/1", "192x192/3", "192x256/1", "192x256/4"]),
    (705, ["256x192/1", "256x128/2", "384x160/1", "384x160/4"]),
])
def test_prefill_on_the_tiles_of_its_plan(layer, t, plan):
    assert _plan(layer["ctx"], t) == plan
    _check(layer, *_prefill(layer, t, gu.workspace(layer["ctx"].ds_prefill_workspace_bytes(t))))


@pytest.mark.parametrize("h,ffn,t,product,plan", [
    (1024, 16384, 583, 2, "384x128/1"), (1024, 16384, 1122, 3, "384x128/10"),      # tiles that no OPT-13B batch takes
    (1536, 16384, 583, 2, "160x256/1"), (1024, 24576, 772, 3, "160x256/12"),
    (4096, 32768, 114, 3, "128x256/15"),
    (1024, 12288, 261, 3, "192x128/16"), (1024, 12288, 387, 3, "256x128/16"),
])
def test_prefill_on_the_tiles_of_other_layers(gpu, h, ffn, t, product, plan):
    layer = _layer(synth.ModelShape(hidden=h, n_heads=h // 128, head_dim=128, ffn=ffn), 4713)
    products = ((h, 3 * h), (h, h), (h, ffn), (ffn, h))
    assert _plan(layer["ctx"], t, products)[product] == plan
    _check(layer, *_prefill(layer, t, gu.workspace(layer["ctx"].ds_prefill_workspace_bytes(t))))


def test_smallest_workspace_runs_on_plans_that_fit_it(gpu):
    """What was enough for ds_linear's plans stays enough, on plans that split less, and a byte less is refused."""
    h, m, t = 1536, 12288, 320
    layer = _layer(synth.ModelShape(hidden=h, n_heads=12, head_dim=128, ffn=m), 4712)
    ctx = layer["ctx"]
    up = lambda v: (v + 255) // 256 * 256
    partials = max(ctx.ds_linear_workspace_bytes(r, k, n) for r in (*range(1, 257), 257, t)
                   for k, n in ((h, 3 * h), (h, h), (h, m), (m, h)))
    least, full = 4 * up(2 * t * h) + up(2 * t * (m + 64)) + up(partials), ctx.ds_prefill_workspace_bytes(t)
    assert least < full
    ws = torch.full((full,), 0x55, dtype=torch.uint8, device="cuda")
    _check(layer, *_prefill(layer, t, ws))
    ws.fill_(0x55)
    _check(layer, *_prefill(layer, t, ws[:least]))
    assert bool((ws[least:] == 0x55).all()), "wrote past the workspace"
    with pytest.raises(binding.DsError):
        _prefill(layer, t, ws[:least - 1])


def _kv_scatter_case(shape, batch):
    """One decoding step; its K and V rows against the product in float64, every other slot of the pool untouched."""
    h, s, n_kv = shape.hidden, shape.head_dim, shape.kv_heads
    kvw, m = n_kv * s, shape.ffn
    ctx = gu.make_ctx(shape)
    g = torch.Generator(device="cuda")
    g.manual_seed(batch)
    draw = lambda *size, std=1.0, mean=0.0: torch.empty(size, dtype=torch.bfloat16, device="cuda").normal_(
        mean, std, generator=g)
    w = {"ln1_g": draw(h, std=0.02, mean=1.0), "ln1_b": draw(h, std=0.02), "w_qkv": draw(h + 2 * kvw, h, std=0.02),
         "b_qkv": draw(h + 2 * kvw, std=0.02), "w_o": draw(h, h, std=0.02), "b_o": draw(h, std=0.02),
         "ln2_g": draw(h, std=0.02, mean=1.0), "ln2_b": draw(h, std=0.02), "w_fc1": draw(m, h, std=0.02),
         "b_fc1": draw(m, std=0.02), "w_fc2": draw(h, m, std=0.02), "b_fc2": draw(h, std=0.02)}
    lw, keep = ctx.pack_weights(w)
    lens = [1 + (7 * i) % 40 for i in range(batch)]
    tables, nblk = synth.make_block_tables([l + 1 for l in lens], 16, 5)
    kc, vc = draw(nblk, n_kv, 16, s), draw(nblk, n_kv, 16, s)
    want_k, want_v = kc.double(), vc.double()
    x, y = draw(batch, h), torch.empty(batch, h, dtype=torch.bfloat16, device="cuda")
    xd = x.double()
    a = (xd - xd.mean(1, keepdim=True)) / torch.sqrt(xd.var(1, unbiased=False, keepdim=True) + 1e-5)
    a = (a * w["ln1_g"].double() + w["ln1_b"].double()).bfloat16().double()    # the rows the product is given
    kv = a @ w["w_qkv"][h:].double().T + w["b_qkv"][h:].double()
    for i, l in enumerate(lens):
        blk = int(tables[i][l // 16])
        want_k[blk, :, l % 16] = kv[i, :kvw].view(n_kv, s)
        want_v[blk, :, l % 16] = kv[i, kvw:].view(n_kv, s)
    ws = gu.workspace(ctx.ds_decode_workspace_bytes(batch, max(lens) + 1))
    ctx.ds_decode_step(lw, x, gu.i32_dev(lens), gu.i32_dev(tables), batch, tables.shape[1], max(lens) + 1, kc, vc, nblk,
                       y, ws)
    torch.cuda.synchronize()
    for got, want in ((kc, want_k), (vc, want_v)):
        # one bf16 rounding of the result (2^-9) and of a on the way to it (another LayerNorm order may flip one)
        assert float((got.double() - want).abs().max()) <= 2.0 ** -7 * float(want.abs().max())


@pytest.mark.parametrize("batch,tile", [(100, (128, 192)), (150, (160, 192)), (180, (192, 192)), (200, (224, 192)),
                                        (250, (256, 160))])
def test_decode_step_scatters_k_and_v_from_unsplit_tiles(gpu, batch, tile):
    """OPT-175B's QKV projection is wide enough to stay unsplit: the tile's own epilogue writes the step's K and V into
    the pages (each sequence's next slot, and nothing else)."""
    shape = synth.ModelShape(hidden=12288, n_heads=96, head_dim=128, ffn=512)
    plan = gu.make_ctx(shape).ds_layer_plan(batch, 12288, 36864)
    assert (plan["tile_rows"], plan["tile_cols"], plan["splits"]) == (*tile, 1)
    _kv_scatter_case(shape, batch)


@pytest.mark.parametrize("heads,n_kv,batch,tile", [(56, 0, 970, (256, 192)), (72, 8, 1810, (256, 192)),
                                                   (16, 8, 4200, (256, 160)), (16, 0, 6000, (256, 160))])
def test_decode_step_scatters_k_and_v_on_both_sides_of_a_cut(gpu, heads, n_kv, batch, tile):
    """QKV on large tiles in whole rounds, the remaining columns - of V, or of K and V - on other tiles."""
    shape = synth.ModelShape(hidden=heads * 128, n_heads=heads, head_dim=128, ffn=512, n_kv_heads=n_kv)
    plan = gu.make_ctx(shape).ds_layer_plan(batch, shape.hidden, shape.qkv_width)
    assert (plan["tile_rows"], plan["tile_cols"]) == tile and 0 < plan["cut_cols"] < shape.qkv_width
    _kv_scatter_case(shape, batch)


@pytest.mark.parametrize("batch", [1, 15, 16, 33, 64, 67, 129])
@pytest.mark.parametrize("heads,head_dim,n_kv", [(4, 64, 0), (6, 128, 2), (8, 128, 0)])
def test_decode_step_scatters_k_and_v_of_small_layers(gpu, heads, head_dim, n_kv, batch):
    """Projections of a few workgroups: unsplit on the ring kernel, with and without a reduce pass, and on tiles."""
    _kv_scatter_case(synth.ModelShape(hidden=heads * head_dim, n_heads=heads, head_dim=head_dim, ffn=256,
                                      n_kv_heads=n_kv), batch)
