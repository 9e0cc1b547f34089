"""The tile GEMM's workgroup order: with 16 or more row tiles the workgroups that run together take 16 x 16 patches,
one block of 8 x 4 tiles per chip partition.  Every output tile has to be computed exactly once, whatever the number
of row and column tiles.  Only whole chunks of 256 tiles are dealt out that way, so every case has at least one."""
import numpy as np
import pytest
import torch

from oracle import ds_oracle as orc
from paper_2401_09670_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,in_f,out_f,tile_cols,tiles_m,tiles_n", [
    (4096, 64, 4096, 256, 16, 16),     # one chunk and nothing else
    (4100, 128, 4104, 160, 17, 26),    # one chunk; a last group of one row tile in the part that is dealt out evenly
    (6100, 192, 7176, 256, 24, 29),    # the second of two chunks runs from a group of 16 row tiles into one of 8
    (5632, 256, 10248, 256, 22, 41),   # ... the third of three into one of 6
    (8200, 192, 8200, 160, 33, 52),    # six chunks, the fourth in two groups; a last group of one row tile
])
def test_linear_many_row_tiles(gpu, rows, in_f, out_f, tile_cols, tiles_m, tiles_n):
    ctx = gu.make_ctx(synth.TINY)
    assert ctx.ds_linear_plan(rows, in_f, out_f) == dict(streaming=False, tile_rows=256, tile_cols=tile_cols, splits=1,
                                                         cut_cols=0)
    assert (tiles_m, tiles_n) == (-(-rows // 256), -(-out_f // tile_cols)) and tiles_m * tiles_n >= 256
    x, w = gu.dev_normal_bits((rows, in_f), 1.0, 11 + rows), gu.dev_normal_bits((out_f, in_f), 0.05, 12 + out_f)
    y = torch.full((rows + 1, out_f), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = gu.workspace(ctx.ds_linear_workspace_bytes(rows, in_f, out_f))
    ctx.ds_linear(x, w, None, None, 0, rows, in_f, out_f, y, ws)
    torch.cuda.synchronize()
    got = gu.to_f64(y)
    ref = orc.linear(gu.to_f64(x), gu.to_f64(w), None)
    assert np.all(got[rows] == 7.0), "wrote past the last row"
    # one bf16 rounding of the result (2^-9) and fp32 sums of at most 256 products, relative to the largest value
    assert float(np.max(np.abs(got[:rows] - ref))) <= 2.0 ** -8 * float(np.max(np.abs(ref)))
