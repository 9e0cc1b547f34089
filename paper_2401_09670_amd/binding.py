"""Binding of libds.so — argument marshalling only: ctypes for contexts, sizes and plans, the module ``_calls``
(``csrc/py_calls.cpp``) for the calls that take tensors.

Every function here has the name and argument order of its C counterpart in
``include/ds.h`` (minus the context, which ``Context`` carries).  Tensors are
torch CUDA tensors used purely as device buffers: the binding passes
``data_ptr()`` and sizes, and the current torch stream as the HIP stream.
The arguments of a decode step take 1.0 us (3.0 with ctypes, and the stream's object came on top: of a small model's
request, ten calls of a few launches each, that was a sixth).
There is no CPU fallback: if the library cannot be loaded, calls raise.
"""
from __future__ import annotations

import ctypes
import os
from types import SimpleNamespace
from typing import Dict, Optional, Tuple

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(PKG_DIR, "libds.so")
CALLS_PATH = os.path.join(PKG_DIR, "_calls.so")

DS_OK = 0
STATIC_SCRATCH_BYTES = 32 << 20   # DS_STATIC_SCRATCH_BYTES of include/ds.h
STATUS_NAMES = {0: "DS_OK", 1: "DS_ERR_INVALID_ARG", 2: "DS_ERR_UNSUPPORTED", 3: "DS_ERR_WORKSPACE",
                4: "DS_ERR_HIP", 5: "DS_ERR_BOUNDS"}
KERNEL_CLASSES = ("layernorm", "gemm", "prefill_attn", "kv_migrate", "skinny_gemm", "decode_attn", "kv_append",
                  "token_io")

# every symbol include/ds.h declares
EXPORTS = ("ds_create", "ds_destroy", "ds_last_error", "ds_set_validate", "ds_prefill_workspace_bytes",
           "ds_decode_workspace_bytes", "ds_prefill", "ds_kv_migrate", "ds_decode_step", "ds_decode_step_static",
           "ds_layernorm",
           "ds_linear_workspace_bytes", "ds_linear_plan", "ds_layer_plan", "ds_linear", "ds_prefill_attention", "ds_decode_attention",
           "ds_embed", "ds_next_token_workspace_bytes", "ds_next_token", "ds_profile_enable", "ds_profile_collect")


class DsError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"{STATUS_NAMES.get(status, status)}: {text}")
        self.status = status


class ModelCfg(ctypes.Structure):
    _fields_ = [("hidden", ctypes.c_int32), ("n_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32),
                ("ffn", ctypes.c_int32), ("block_size", ctypes.c_int32), ("ln_eps", ctypes.c_float),
                ("n_kv_heads", ctypes.c_int32)]


class LayerWeights(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in
                ("ln1_g", "ln1_b", "w_qkv", "b_qkv", "w_o", "b_o", "ln2_g", "ln2_b",
                 "w_fc1", "b_fc1", "w_fc2", "b_fc2")]


# the entry points that take tensors: their library functions are called through the module _calls
TENSOR_CALLS = ("ds_prefill", "ds_kv_migrate", "ds_decode_step", "ds_decode_step_static", "ds_layernorm", "ds_linear",
                "ds_prefill_attention", "ds_decode_attention", "ds_embed", "ds_next_token")

_lib = None


def is_built() -> bool:
    """Whether the library and the module that calls it are there."""
    return os.path.exists(LIB_PATH) and os.path.exists(CALLS_PATH)


def load_library() -> ctypes.CDLL:
    """Load libds.so and ``_calls`` (built in-tree by ``build``); raises if either is absent."""
    global _lib
    if _lib is not None:
        return _lib
    for path in (LIB_PATH, CALLS_PATH):
        if not os.path.exists(path):
            raise RuntimeError(f"{path} is missing: build it with __graft_entry__.build() "
                               "(there is no fallback path)")
    # torch ships a HIP runtime of its own under the same library name: it has to be the one in the process
    # before libds.so asks for it, or torch later finds the system's copy loaded in its place (seen as a
    # segmentation fault at torch's first GPU call when this library was loaded first)
    import torch  # noqa: F401
    from . import _calls
    lib = ctypes.CDLL(LIB_PATH)
    vp, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
    lib.ds_create.argtypes = [ctypes.POINTER(ModelCfg), ctypes.POINTER(vp)]
    lib.ds_create.restype = ctypes.c_int
    lib.ds_destroy.argtypes = [vp]
    lib.ds_destroy.restype = None
    lib.ds_last_error.argtypes = [vp]
    lib.ds_last_error.restype = ctypes.c_char_p
    lib.ds_set_validate.argtypes = [vp, i32]
    lib.ds_set_validate.restype = ctypes.c_int
    lib.ds_prefill_workspace_bytes.argtypes = [vp, i32]
    lib.ds_prefill_workspace_bytes.restype = sz
    lib.ds_decode_workspace_bytes.argtypes = [vp, i32, i32]
    lib.ds_decode_workspace_bytes.restype = sz
    lib.ds_prefill.argtypes = [vp, ctypes.POINTER(LayerWeights), vp, vp, i32, i32, i32, vp, vp, vp, vp, sz, vp]
    lib.ds_prefill.restype = ctypes.c_int
    lib.ds_kv_migrate.argtypes = [vp, vp, vp, vp, i32, i32, i32, vp, i32, vp, vp, i32, vp]
    lib.ds_kv_migrate.restype = ctypes.c_int
    lib.ds_decode_step.argtypes = [vp, ctypes.POINTER(LayerWeights), vp, vp, vp, i32, i32, i32, vp, vp, i32,
                                   vp, vp, sz, vp]
    lib.ds_decode_step.restype = ctypes.c_int
    lib.ds_decode_step_static.argtypes = [vp, ctypes.POINTER(LayerWeights), vp, vp, vp, i32, i32, i32, vp, vp, i32,
                                          vp, vp]
    lib.ds_decode_step_static.restype = ctypes.c_int
    lib.ds_layernorm.argtypes = [vp, vp, vp, vp, i32, vp, vp]
    lib.ds_layernorm.restype = ctypes.c_int
    lib.ds_linear_workspace_bytes.argtypes = [vp, i32, i32, i32]
    lib.ds_linear_workspace_bytes.restype = sz
    for plan in (lib.ds_linear_plan, lib.ds_layer_plan):
        plan.argtypes = [vp, i32, i32, i32] + [ctypes.POINTER(ctypes.c_int32)] * 5
        plan.restype = ctypes.c_int
    lib.ds_linear.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, i32, vp, vp, sz, vp]
    lib.ds_linear.restype = ctypes.c_int
    lib.ds_prefill_attention.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, vp, vp]
    lib.ds_prefill_attention.restype = ctypes.c_int
    lib.ds_decode_attention.argtypes = [vp, vp, vp, vp, i32, i32, i32, vp, vp, i32, vp, vp, sz, vp]
    lib.ds_decode_attention.restype = ctypes.c_int
    lib.ds_embed.argtypes = [vp, vp, vp, vp, i32, vp, i32, i32, vp, vp]
    lib.ds_embed.restype = ctypes.c_int
    lib.ds_next_token_workspace_bytes.argtypes = [vp, i32, i32]
    lib.ds_next_token_workspace_bytes.restype = sz
    lib.ds_next_token.argtypes = [vp, vp, vp, i32, vp, vp, vp, i32, vp, vp, vp, sz, vp]
    lib.ds_next_token.restype = ctypes.c_int
    lib.ds_profile_enable.argtypes = [vp, i32]
    lib.ds_profile_enable.restype = ctypes.c_int
    lib.ds_profile_collect.argtypes = [vp, ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_int64)]
    lib.ds_profile_collect.restype = ctypes.c_int
    lib.tensor_calls = SimpleNamespace(**{
        n: _calls.bind(n, ctypes.cast(getattr(lib, n), vp).value, LayerWeights) for n in TENSOR_CALLS})
    _lib = lib
    return lib


def _ptr(t) -> Optional[int]:
    """Device (or NULL) pointer of a torch tensor."""
    if t is None:
        return None
    return t.data_ptr()


def _stream() -> int:
    """The current torch stream of the current device (0: the default stream)."""
    import torch
    if not torch.cuda.is_initialized():
        return torch.cuda.current_stream().cuda_stream
    return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())


class Context:
    """``ds_ctx`` for one layer shape; methods mirror the C entry points."""

    def __init__(self, hidden: int, n_heads: int, head_dim: int, ffn: int, block_size: int = 16,
                 ln_eps: float = 1e-5, n_kv_heads: int = 0):
        self.lib = load_library()
        self.calls = self.lib.tensor_calls
        self.cfg = ModelCfg(hidden, n_heads, head_dim, ffn, block_size, ln_eps, n_kv_heads)
        self.handle = ctypes.c_void_p()
        st = self.lib.ds_create(ctypes.byref(self.cfg), ctypes.byref(self.handle))
        if st != DS_OK:
            self.handle = ctypes.c_void_p()
            raise DsError(st, "ds_create rejected the configuration")

    def close(self):
        if getattr(self, "handle", None) and self.handle.value:
            self.lib.ds_destroy(self.handle)
            self.handle = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _check(self, st: int):
        if st != DS_OK:
            raise DsError(st, self.lib.ds_last_error(self.handle).decode())

    @staticmethod
    def pack_weights(w: Dict[str, "object"]) -> Tuple[LayerWeights, dict]:
        """dict of device tensors (missing / None bias = NULL) -> (struct, keep-alive dict)."""
        lw = LayerWeights()
        for name, _ in LayerWeights._fields_:
            setattr(lw, name, _ptr(w.get(name)))
        return lw, w

    def ds_set_validate(self, on: bool):
        self._check(self.lib.ds_set_validate(self.handle, 1 if on else 0))

    # ---- sizes ----
    def ds_prefill_workspace_bytes(self, max_tokens: int) -> int:
        return self.lib.ds_prefill_workspace_bytes(self.handle, max_tokens)

    def ds_decode_workspace_bytes(self, max_batch: int, max_ctx: int) -> int:
        return self.lib.ds_decode_workspace_bytes(self.handle, max_batch, max_ctx)

    def ds_linear_workspace_bytes(self, rows: int, in_f: int, out_f: int) -> int:
        return self.lib.ds_linear_workspace_bytes(self.handle, rows, in_f, out_f)

    # ---- the three calls of the path ----
    def ds_prefill(self, weights: LayerWeights, x, cu_seqlens, B: int, t: int, max_seqlen: int, y, k_out, v_out,
                   workspace):
        self._check(self.calls.ds_prefill(self.handle.value, weights, x, cu_seqlens, B, t, max_seqlen, y, k_out,
                                          v_out, workspace, workspace, _stream()))

    def ds_kv_migrate(self, k_src, v_src, cu_seqlens, B: int, t: int, max_seqlen: int, block_tables,
                      max_blocks_per_seq: int, k_cache, v_cache, num_blocks: int):
        self._check(self.calls.ds_kv_migrate(self.handle.value, k_src, v_src, cu_seqlens, B, t, max_seqlen,
                                             block_tables, max_blocks_per_seq, k_cache, v_cache, num_blocks,
                                             _stream()))

    def ds_decode_step(self, weights: LayerWeights, x, ctx_lens, block_tables, B: int, max_blocks_per_seq: int,
                       max_ctx: int, k_cache, v_cache, num_blocks: int, y, workspace):
        self._check(self.calls.ds_decode_step(self.handle.value, weights, x, ctx_lens, block_tables, B,
                                              max_blocks_per_seq, max_ctx, k_cache, v_cache, num_blocks, y,
                                              workspace, workspace, _stream()))

    def ds_decode_step_static(self, weights: LayerWeights, x, ctx_lens, block_tables, B: int,
                              max_blocks_per_seq: int, max_ctx: int, k_cache, v_cache, num_blocks: int, y):
        self._check(self.calls.ds_decode_step_static(self.handle.value, weights, x, ctx_lens, block_tables, B,
                                                     max_blocks_per_seq, max_ctx, k_cache, v_cache, num_blocks, y,
                                                     _stream()))

    # ---- single steps ----
    def ds_layernorm(self, x, gamma, beta, rows: int, out):
        self._check(self.calls.ds_layernorm(self.handle.value, x, gamma, beta, rows, out, _stream()))

    def ds_linear_plan(self, rows: int, in_f: int, out_f: int) -> dict:
        return self._plan(self.lib.ds_linear_plan, rows, in_f, out_f)

    def ds_layer_plan(self, rows: int, in_f: int, out_f: int) -> dict:
        return self._plan(self.lib.ds_layer_plan, rows, in_f, out_f)

    def _plan(self, query, rows: int, in_f: int, out_f: int) -> dict:
        v = [ctypes.c_int32() for _ in range(5)]
        self._check(query(self.handle, rows, in_f, out_f, *[ctypes.byref(a) for a in v]))
        return dict(streaming=bool(v[0].value), tile_rows=v[1].value, tile_cols=v[2].value, splits=v[3].value,
                    cut_cols=v[4].value)

    def ds_linear(self, x, w, bias, residual, relu: int, rows: int, in_f: int, out_f: int, y, workspace=None):
        self._check(self.calls.ds_linear(self.handle.value, x, w, bias, residual, relu, rows, in_f, out_f, y,
                                         workspace, workspace, _stream()))

    def ds_prefill_attention(self, q, k, v, cu_seqlens, B: int, t: int, max_seqlen: int, o):
        self._check(self.calls.ds_prefill_attention(self.handle.value, q, k, v, cu_seqlens, B, t, max_seqlen, o,
                                                    _stream()))

    def ds_decode_attention(self, q, kv_lens, block_tables, B: int, max_blocks_per_seq: int, max_kv_len: int,
                            k_cache, v_cache, num_blocks: int, o, workspace=None):
        self._check(self.calls.ds_decode_attention(self.handle.value, q, kv_lens, block_tables, B,
                                                   max_blocks_per_seq, max_kv_len, k_cache, v_cache, num_blocks, o,
                                                   workspace, workspace, _stream()))

    # ---- the two ends of the token loop ----
    def ds_embed(self, token_ids, positions, tok_emb, vocab: int, pos_emb, n_pos: int, rows: int, x):
        self._check(self.calls.ds_embed(self.handle.value, token_ids, positions, tok_emb, vocab, pos_emb, n_pos,
                                        rows, x, _stream()))

    def ds_next_token_workspace_bytes(self, rows: int, vocab: int) -> int:
        return self.lib.ds_next_token_workspace_bytes(self.handle, rows, vocab)

    def ds_next_token(self, x, row_index, rows: int, ln_g, ln_b, w_vocab, vocab: int, next_token, best_logit,
                      workspace):
        self._check(self.calls.ds_next_token(self.handle.value, x, row_index, rows, ln_g, ln_b, w_vocab, vocab,
                                             next_token, best_logit, workspace, workspace, _stream()))

    # ---- timing ----
    def ds_profile_enable(self, on: bool):
        self._check(self.lib.ds_profile_enable(self.handle, 1 if on else 0))

    def ds_profile_collect(self):
        n = len(KERNEL_CLASSES)
        ms = (ctypes.c_double * n)()
        cnt = (ctypes.c_int64 * n)()
        self._check(self.lib.ds_profile_collect(self.handle, ms, cnt))
        return {k: (ms[i], cnt[i]) for i, k in enumerate(KERNEL_CLASSES)}
