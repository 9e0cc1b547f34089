"""Workspace sizes on the host: the same whatever was asked before, and cheap for a size that is new to a context (each
ds_prefill or ds_decode_step checks its workspace, and a ragged batch brings a new size almost every call)."""
import random
import time

import pytest

from paper_2401_09670_amd import binding

SHAPES = {"tiny": (256, 4, 64, 1024, 0), "opt13b": (5120, 40, 128, 20480, 0), "gqa": (8192, 64, 128, 32768, 8)}


def _ctx(name):
    h, n, s, m, n_kv = SHAPES[name]
    return binding.Context(h, n, s, m, n_kv_heads=n_kv)


@pytest.mark.parametrize("name", SHAPES)
def test_sizes_do_not_depend_on_what_was_asked_before(name):
    counts = [1, 64, 65, 96, 97, 129, 256, 257, 319, 320, 321, 700, 4096, 4097, 4161, 65536, 65599, 65600, 70001]
    random.Random(5).shuffle(counts)
    warm = _ctx(name)
    for n in counts:
        assert warm.ds_prefill_workspace_bytes(n) == _ctx(name).ds_prefill_workspace_bytes(n)
        if n < 5000:
            assert warm.ds_decode_workspace_bytes(n, 700) == _ctx(name).ds_decode_workspace_bytes(n, 700)


def test_a_new_size_does_not_go_through_all_smaller_ones_again():
    counts = list(range(1000, 4000, 50))

    def seconds(contexts):
        start = time.perf_counter()
        for ctx, n in zip(contexts, counts):
            ctx.ds_prefill_workspace_bytes(n)
        return time.perf_counter() - start

    warm = _ctx("opt13b")
    warm.ds_prefill_workspace_bytes(4096)
    fresh = [_ctx("opt13b") for _ in counts]
    assert seconds([warm] * len(counts)) < 0.25 * seconds(fresh)      # (a fiftieth; with no memory of rows the same)
