"""Plans of the products inside ds_prefill and ds_decode_step (host only): what any of them must satisfy, and that the
workspaces the library asks for hold their partial sums."""
import pytest

from paper_2401_09670_amd import binding

SHAPES = {"tiny": (256, 4, 64, 1024, 0), "opt13b": (5120, 40, 128, 20480, 0), "opt66b": (9216, 72, 128, 36864, 0),
          "opt175b": (12288, 96, 128, 49152, 0), "gqa": (8192, 64, 128, 32768, 8)}
TILES = {(64, 128), (96, 192), (128, 128), (128, 192), (128, 256), (160, 192), (160, 256), (192, 128), (192, 192),
         (192, 256), (224, 192), (256, 128), (256, 160), (256, 192), (256, 256), (288, 192), (320, 192), (384, 128),
         (384, 160)}


def _ctx(name):
    h, n, s, m, n_kv = SHAPES[name]
    return binding.Context(h, n, s, m, n_kv_heads=n_kv)


def _products(name):
    h, n, s, m, n_kv = SHAPES[name]
    return ((h, (n + 2 * (n_kv or n)) * s), (h, h), (h, m), (m, h))


def _partials(plan, rows, out_f):
    return 4 * plan["splits"] * rows * out_f if plan["splits"] > 1 else 0


@pytest.mark.parametrize("name", SHAPES)
def test_layer_plan_invariants(name):
    ctx = _ctx(name)
    for rows in (65, 96, 97, 128, 129, 160, 193, 256, 257, 289, 321, 512, 700, 1023, 2048, 2985, 4096):
        for k, n in _products(name):
            p = ctx.ds_layer_plan(rows, k, n)
            if p["streaming"]:
                assert rows <= 128 and ctx.ds_linear_plan(rows, k, n)["streaming"]
                continue
            assert (p["tile_rows"], p["tile_cols"]) in TILES
            tiles = -(-rows // p["tile_rows"]) * -(-n // p["tile_cols"])
            if p["splits"] > 1:
                assert tiles * p["splits"] <= 256 and k // 64 // p["splits"] >= 6 and p["cut_cols"] == 0
            if p["cut_cols"]:      # whole rounds before the cut, columns left behind it
                assert 0 < p["cut_cols"] < n and p["cut_cols"] % p["tile_cols"] == 0
                assert -(-rows // p["tile_rows"]) * (p["cut_cols"] // p["tile_cols"]) % 256 == 0


def test_small_products_and_the_out_projection_are_reported_as_a_layer_runs_them():
    """A small product stays unsplit in a layer; LayerNorm-2 rides in a reduce pass, so the out-projection is not taken by
    the unsplit kernel (64 columns a workgroup) that ds_linear has for so many columns."""
    ctx = _ctx("tiny")
    assert ctx.ds_linear_plan(2, 1024, 256)["splits"] == 8 and ctx.ds_layer_plan(2, 1024, 256)["splits"] == 1
    ctx, out = _ctx("opt175b"), (12288, 12288)
    assert ctx.ds_linear_plan(8, *out)["splits"] == 1 and ctx.ds_layer_plan(8, *out)["splits"] > 1


def test_outside_their_rows_large_layers_and_single_products_plan_alike():
    ctx = _ctx("opt13b")
    for rows in (1, 17, 64, 4097, 16384):
        for k, n in _products("opt13b"):
            assert ctx.ds_layer_plan(rows, k, n) == ctx.ds_linear_plan(rows, k, n)


@pytest.mark.parametrize("name", SHAPES)
def test_workspaces_hold_the_partial_sums_of_every_smaller_call(name):
    ctx = _ctx(name)
    h, n, s, m, n_kv = SHAPES[name]
    wide = (n + 2 * (n_kv or n)) * s
    for most in (70, 129, 300, 1000):
        pre, dec = ctx.ds_prefill_workspace_bytes(most), ctx.ds_decode_workspace_bytes(most, 64)
        for rows in range(65, most + 1, 3):
            need = max(_partials(ctx.ds_layer_plan(rows, k, o), rows, o) for k, o in _products(name))
            assert pre >= rows * 2 * (4 * h + m + 64) + need
            assert dec >= rows * 2 * (3 * h + wide + m) + need


@pytest.mark.parametrize("name,largest", [("opt13b", 128), ("opt66b", 92), ("opt175b", 72), ("gqa", 124)])
def test_decode_workspace_says_what_the_static_array_takes(name, largest):
    """The largest batch that ds_decode_step_static accepts is the largest whose reported workspace fits its array: what
    the plans of ds_linear need, not what the faster ones of a layer would use."""
    h, n, s, m, n_kv = SHAPES[name]
    wide, up = (n + 2 * (n_kv or n)) * s, lambda v: (v + 255) // 256 * 256
    ctx = _ctx(name)

    def least(batch):       # (without attention partials: none at 16 tokens)
        partials = max(ctx.ds_linear_workspace_bytes(r, k, o) for r in range(1, batch + 1) for k, o in _products(name))
        return sum(up(2 * batch * f) for f in (h, h, h, wide, m)) + up(partials)

    assert least(largest) <= binding.STATIC_SCRATCH_BYTES < least(largest + 1)
    assert ctx.ds_decode_workspace_bytes(largest, 16) <= binding.STATIC_SCRATCH_BYTES
    assert ctx.ds_decode_workspace_bytes(largest + 1, 16) > binding.STATIC_SCRATCH_BYTES


@pytest.mark.parametrize("name,product,rows,lost", [
    # tile and splits of plans that were measured slower than what ds_linear runs, or than others of the layer's own
    ("opt13b", 1, (129, 160, 161, 192), ((192, 128), 5)), ("opt13b", 1, (193, 208, 225, 256), ((256, 128), 5)),
    ("gqa", 3, (88, 96, 128), ((128, 256), 8)), ("gqa", 3, (129, 160), ((160, 256), 8)), ("gqa", 3, (161, 192), ((192, 256), 8)),
])
def test_plans_that_measured_slower_are_not_taken(name, product, rows, lost):
    ctx = _ctx(name)
    for r in rows:
        p = ctx.ds_layer_plan(r, *_products(name)[product])
        assert ((p["tile_rows"], p["tile_cols"]), p["splits"]) != lost
        if name == "opt13b":
            assert p == ctx.ds_linear_plan(r, *_products(name)[product])


def test_a_cut_is_taken_where_it_pays():
    """A second launch costs more than the model's sum: 279 us cut, 269 not (OPT-66B out-projection, 2048 rows); 746 and 797
    (its QKV)."""
    ctx = _ctx("opt66b")
    (k, qkv), out = _products("opt66b")[0], _products("opt66b")[1]
    assert ctx.ds_layer_plan(2048, *out)["cut_cols"] == 0 < ctx.ds_layer_plan(2048, k, qkv)["cut_cols"]
    for name in ("opt66b", "opt175b"):
        assert _ctx(name).ds_layer_plan(512, *_products(name)[0])["cut_cols"] == 0
