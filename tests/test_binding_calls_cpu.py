"""The module through which the binding calls the library: what reaches the C side of each argument, and what is
refused, with ctypes callbacks in the library's place (the types are those of the entry points' ctypes signatures)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2401_09670_amd import binding

binding.load_library()  # (says what to build, if anything)
from paper_2401_09670_amd import _calls  # noqa: E402

VP, I32, SZ = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t


def _entry(name, seen, status=0):
    """The entry point `name` in a library whose function only notes its arguments."""
    types = getattr(binding.load_library(), name).argtypes
    plain = [VP if t not in (VP, I32, SZ) else t for t in types]
    fn = ctypes.CFUNCTYPE(ctypes.c_int, *plain)(lambda *a: seen.append(a) or status)
    call = _calls.bind(name, ctypes.cast(fn, VP).value, binding.LayerWeights)
    return call, types, fn


@pytest.mark.parametrize("name", binding.TENSOR_CALLS)
@pytest.mark.parametrize("with_tensors", [True, False])
def test_every_argument_reaches_its_place(name, with_tensors):
    seen = []
    call, types, _keep = _entry(name, seen, status=3)
    weights, args, want = binding.LayerWeights(), [], []
    for i, t in enumerate(types):
        if i == 0 or i == len(types) - 1:                  # the context and the stream: addresses
            args.append((1 << 47) + i if with_tensors else None)
            want.append(args[-1])
        elif t is I32:
            args.append(-7 - i)
            want.append(-7 - i)
        elif t is SZ:                                      # the bytes of the workspace before it
            args.append(args[-1])
            want.append(args[-1].nbytes if with_tensors else 0)
        elif t is VP:
            args.append(torch.zeros(3 + i, dtype=torch.bfloat16) if with_tensors else None)
            want.append(args[-1].data_ptr() if with_tensors else None)
        else:
            args.append(weights)
            want.append(ctypes.addressof(weights))
    assert call(*args) == 3
    assert list(seen[0]) == want
    with pytest.raises(TypeError):
        call(*args[:-1])
    with pytest.raises(TypeError):
        call(*args, 0)
    assert len(seen) == 1


@pytest.mark.parametrize("rows,want", [
    (True, 1), (np.int64(5), 5), (np.int32(-1), -1), (torch.tensor(9), 9), (ctypes.c_int32(11), 11), (0, 0),
    (2 ** 31 - 1, 2 ** 31 - 1), (-2 ** 31, -2 ** 31), (2 ** 32 + 6, 6),
])
def test_whole_numbers_as_ctypes_takes_them(rows, want):
    seen = []
    call, _, _keep = _entry("ds_layernorm", seen)
    assert call(None, None, None, None, rows, None, 0) == 0
    assert seen[0][4] == want


@pytest.mark.parametrize("args", [
    (None, None, None, None, 1.0, None, 0), (None, None, None, None, "1", None, 0),
    (None, None, None, None, None, None, 0), (None, 4096, None, None, 1, None, 0),
    (None, np.zeros(4), None, None, 1, None, 0), (None, None, None, None, 1, None, "0"),
    (None, None, None, None, ctypes.c_float(1.0), None, 0), (None, None, None, None, ctypes.c_int64(1), None, 0),
])
def test_other_arguments_are_refused(args):
    seen = []
    call, _, _keep = _entry("ds_layernorm", seen)
    with pytest.raises((TypeError, AttributeError)):
        call(*args)
    assert not seen


@pytest.mark.parametrize("weights", [None, 0, (ctypes.c_void_p * 12)(), np.zeros(12, np.int64)])
def test_weights_are_the_struct(weights):
    seen = []
    call, _, _keep = _entry("ds_decode_step_static", seen)
    with pytest.raises(TypeError):
        call(None, weights, None, None, None, 1, 1, 1, None, None, 1, None, None)
    assert not seen


def test_an_unknown_name_is_refused():
    with pytest.raises(KeyError):
        _calls.bind("ds_no_such_call", 1, binding.LayerWeights)
