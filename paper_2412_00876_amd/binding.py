"""Thin binding of libdllava.so: argument marshalling only.

The functions below say through ctypes what each call takes; at the end of the module they are bound to their native forms
(native/calls.cpp), which convert the same arguments without ctypes and leave whatever they do not know to them.  Where the native
forms are not there, or were built for another torch, the functions stay what they are: the same calls, a few microseconds of
host time longer each.

Every function has the name and argument order of its C entry point (include/dllava.h); tensors are
torch tensors used purely as device buffers (data_ptr), and the stream defaults to torch's current
stream.  A non-zero status raises DllavaError with the library's message.  Nothing here computes:
if the shared library is missing the import fails.
"""
from __future__ import annotations

import ctypes as C
import functools
import os
import warnings
from typing import Optional

import torch

_LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "lib", "libdllava.so")

F32, BF16 = 0, 1
MODE_TOPK, MODE_THRESHOLD, MODE_THRESHOLD_KEEP_LAST = 0, 1, 2
LAUNCH_DECODE_WAVES, LAUNCH_DECODE_SPLITS, LAUNCH_PREFILL_WAVES, LAUNCH_SCORE_TILE, LAUNCH_QKV_TILE, LAUNCH_PREFILL_BLOCKS = 0, 1, 2, 3, 4, 5
LAUNCH_SELECT_LAUNCHES = 6
LAUNCH_LINEAR_TILE = 7
PAGE_SIZE = 16


class DllavaError(RuntimeError):
    def __init__(self, status: int, msg: str):
        super().__init__(f"dllava status {status}: {msg}")
        self.status = status


class _KvCache(C.Structure):
    _fields_ = [("pages", C.c_void_p), ("block_table", C.c_void_p), ("cache_len", C.c_void_p),
                ("n_pages", C.c_int32), ("max_pages_per_seq", C.c_int32), ("page_size", C.c_int32),
                ("H", C.c_int32), ("Dh", C.c_int32), ("dtype", C.c_int32)]


class _VitBlock(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("ln1_g", "ln1_b", "Wqkv", "bqkv", "Wo", "bo", "ln2_g", "ln2_b",
                                          "Wfc1", "bfc1", "Wfc2", "bfc2")]


PREDICTOR_MAX_BLOCKS = 4


class _Predictor(C.Structure):
    _fields_ = [("d", C.c_int64), ("n_blocks", C.c_int32), ("W_in", C.c_void_p), ("b_in", C.c_void_p),
                ("blocks", _VitBlock * PREDICTOR_MAX_BLOCKS),
                ("W_h1", C.c_void_p), ("b_h1", C.c_void_p), ("W_h2", C.c_void_p), ("b_h2", C.c_void_p),
                ("W_h3", C.c_void_p), ("b_h3", C.c_void_p)]


def _load() -> C.CDLL:
    if not os.path.exists(_LIB_PATH):
        raise ImportError(f"{_LIB_PATH} is missing: build it with `python -m paper_2412_00876_amd.build` "
                          "(there is no fallback path)")
    lib = C.CDLL(_LIB_PATH)
    vp, i32, i64, f32, sz = C.c_void_p, C.c_int32, C.c_int64, C.c_float, C.c_size_t
    lib.dllava_version.restype = C.c_int
    lib.dllava_version.argtypes = []
    lib.dllava_last_error.restype = C.c_char_p
    lib.dllava_last_error.argtypes = []
    lib.dllava_set_launch_override.restype = C.c_int
    lib.dllava_set_launch_override.argtypes = [C.c_int, C.c_int]
    lib.dllava_score.restype = C.c_int
    lib.dllava_score.argtypes = [vp, i64, i64, i32, vp, vp, vp, i64, i64, vp, vp, vp, vp, C.c_int, vp, vp, sz, vp]
    lib.dllava_score_workspace.restype = sz
    lib.dllava_score_workspace.argtypes = [i64, i64, i64, C.c_int]
    lib.dllava_select_compact.restype = C.c_int
    lib.dllava_select_compact.argtypes = [vp, i32, vp, vp, vp, i64, C.c_int, C.c_double, f32, vp, vp, i64, vp, vp, vp, vp,
                                          C.POINTER(_KvCache), vp, vp, vp, vp, C.c_int, vp, sz, vp]
    lib.dllava_select_compact_workspace.restype = sz
    lib.dllava_select_compact_workspace.argtypes = [i32, i64]
    lib.dllava_prefill_attn.restype = C.c_int
    lib.dllava_prefill_attn.argtypes = [vp, vp, vp, C.POINTER(_KvCache), i32, vp, i64, i32, i32, f32, vp, C.c_int, vp]
    lib.dllava_decode_attn_append.restype = C.c_int
    lib.dllava_decode_attn_append.argtypes = [vp, vp, vp, i32, vp, f32, vp, C.POINTER(_KvCache), f32, vp, vp, vp,
                                              vp, sz, vp]
    lib.dllava_decode_attn_append_static.restype = C.c_int
    lib.dllava_decode_attn_append_static.argtypes = [vp, vp, vp, i32, vp, f32, vp, C.POINTER(_KvCache), f32, vp, vp, vp, vp]
    lib.dllava_decode_workspace.restype = sz
    lib.dllava_decode_workspace.argtypes = [i32, i32, i32, i32]
    lib.dllava_decode_step.restype = C.c_int
    lib.dllava_decode_step.argtypes = [vp, i64, i64, i64, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, i32, f32,
                                       C.POINTER(_KvCache), f32, vp, vp, vp, vp, vp, sz, vp]
    lib.dllava_decode_step_workspace.restype = sz
    lib.dllava_decode_step_workspace.argtypes = [i32, i32, i32, i32, i64, i64, C.c_int]
    lib.dllava_decode_commit.restype = C.c_int
    lib.dllava_decode_commit.argtypes = [vp, vp, vp, vp, i32, f32, C.POINTER(_KvCache), vp, vp, vp]
    lib.dllava_qkv_project.restype = C.c_int
    lib.dllava_qkv_project.argtypes = [vp, i64, i64, i64, i32, vp, vp, vp, vp, vp, f32, vp, C.POINTER(_KvCache), vp,
                                       C.c_int, vp]
    lib.dllava_predict.restype = C.c_int
    lib.dllava_predict.argtypes = [vp, i64, i64, i32, vp, vp, vp, C.POINTER(_Predictor), C.c_int, vp, vp, sz, vp]
    lib.dllava_predict_workspace.restype = sz
    lib.dllava_predict_workspace.argtypes = [i64, i32, i32]
    lib.dllava_compact.restype = C.c_int
    lib.dllava_compact.argtypes = [i32, vp, vp, vp, i64, vp, vp, i64, vp, vp, vp, vp, C.POINTER(_KvCache), vp, C.c_int, vp]
    lib.dllava_masked_attn.restype = C.c_int
    lib.dllava_masked_attn.argtypes = [vp, vp, vp, i32, vp, i64, i32, i32, f32, vp, vp, C.c_int, vp, sz, vp]
    lib.dllava_masked_attn_workspace.restype = sz
    lib.dllava_masked_attn_workspace.argtypes = [i64, i32]
    lib.dllava_linear.restype = C.c_int
    lib.dllava_linear.argtypes = [vp, i64, i64, i64, vp, vp, i64, C.c_int, vp, vp, i64, C.c_int, vp]
    lib.dllava_layer_norm.restype = C.c_int
    lib.dllava_layer_norm.argtypes = [vp, i64, vp, vp, vp, C.c_int, vp]
    lib.dllava_linear_few.restype = C.c_int
    lib.dllava_linear_few.argtypes = [vp, i64, i64, i64, vp, vp, i64, C.c_int, vp, vp, i64, C.c_int, vp, sz, vp]
    lib.dllava_linear_few_workspace.restype = sz
    lib.dllava_linear_few_workspace.argtypes = [i64, i64]
    lib.dllava_qkv_few.restype = C.c_int
    lib.dllava_qkv_few.argtypes = [vp, i64, i64, i64, vp, vp, vp, i32, i32, vp, f32, vp, vp, vp, C.c_int, vp, sz, vp]
    lib.dllava_gated_few.restype = C.c_int
    lib.dllava_gated_few.argtypes = [vp, i64, i64, i64, vp, vp, i64, vp, i64, C.c_int, vp, sz, vp]
    lib.dllava_decode_proj_workspace.restype = sz
    lib.dllava_decode_proj_workspace.argtypes = [i64, i64]
    lib.dllava_rope.restype = C.c_int
    lib.dllava_rope.argtypes = [vp, vp, i64, i32, i32, f32, C.c_int, vp]
    lib.dllava_rms_norm.restype = C.c_int
    lib.dllava_rms_norm.argtypes = [vp, i64, i64, i64, vp, f32, vp, i64, C.c_int, vp]
    lib.dllava_span_attn.restype = C.c_int
    lib.dllava_span_attn.argtypes = [vp, vp, vp, i32, vp, i64, i32, i32, f32, vp, C.c_int, vp]
    return lib


_lib = _load()
EXPORTS = ("dllava_version", "dllava_last_error", "dllava_set_launch_override", "dllava_score", "dllava_score_workspace",
           "dllava_select_compact", "dllava_select_compact_workspace", "dllava_prefill_attn",
           "dllava_decode_attn_append", "dllava_decode_attn_append_static", "dllava_decode_workspace", "dllava_qkv_project",
           "dllava_decode_step", "dllava_decode_step_workspace", "dllava_decode_commit",
           "dllava_predict", "dllava_predict_workspace", "dllava_linear", "dllava_layer_norm", "dllava_span_attn",
           "dllava_masked_attn", "dllava_masked_attn_workspace", "dllava_compact", "dllava_rms_norm", "dllava_linear_few",
           "dllava_linear_few_workspace", "dllava_rope", "dllava_qkv_few", "dllava_gated_few",
           "dllava_decode_proj_workspace")


def lib() -> C.CDLL:
    return _lib


def dtype_code(t: torch.dtype) -> int:
    if t == torch.float32:
        return F32
    if t == torch.bfloat16:
        return BF16
    raise TypeError(f"unsupported dtype {t}")


def _p(t: Optional[torch.Tensor]) -> Optional[int]:
    return None if t is None else t.data_ptr()


def _stream(stream) -> Optional[int]:
    if stream is None:
        # torch's current stream of the current device, without building a Stream object for it (2.9 us per call; 0.3 us)
        stream = torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())
    elif hasattr(stream, "cuda_stream"):
        stream = stream.cuda_stream
    return stream or None


def _check(rc: int) -> None:
    if rc != 0:
        raise DllavaError(rc, _lib.dllava_last_error().decode())


def _ws(workspace: Optional[torch.Tensor]):
    if workspace is None:
        return None, 0
    return workspace.data_ptr(), workspace.numel() * workspace.element_size()


class KVCache:
    """Host-side descriptor (dllava_kv_cache) over caller-owned device tensors."""

    def __init__(self, pages: torch.Tensor, block_table: torch.Tensor, cache_len: torch.Tensor):
        n_pages, two, H, ps, Dh = pages.shape
        assert two == 2 and pages.is_contiguous() and block_table.is_contiguous()
        assert block_table.dtype == torch.int32 and cache_len.dtype == torch.int32
        self.pages, self.block_table, self.cache_len = pages, block_table, cache_len
        self.H, self.Dh, self.page_size = H, Dh, ps
        self.B, self.max_pages_per_seq = block_table.shape
        self.c = _KvCache(pages.data_ptr(), block_table.data_ptr(), cache_len.data_ptr(), n_pages,
                          self.max_pages_per_seq, ps, H, Dh, dtype_code(pages.dtype))

    @property
    def ref(self):
        return C.byref(self.c)


class Predictor:
    """Host-side descriptor (dllava_predictor) over caller-owned device tensors.

    `weights` maps the struct's field names to tensors (or None for an optional vector); `blocks` is a list of such
    maps, one per transformer block.  The tensors are kept alive by this object.
    """

    def __init__(self, d: int, weights: dict, blocks: list):
        assert len(blocks) <= PREDICTOR_MAX_BLOCKS
        self._keep = (weights, blocks)
        self.n_blocks = len(blocks)
        self.c = _Predictor()
        self.c.d, self.c.n_blocks = d, len(blocks)
        for name in ("W_in", "b_in", "W_h1", "b_h1", "W_h2", "b_h2", "W_h3", "b_h3"):
            setattr(self.c, name, _p(weights.get(name)))
        for i, blk in enumerate(blocks):
            for name, _ in _VitBlock._fields_:
                setattr(self.c.blocks[i], name, _p(blk.get(name)))

    @property
    def ref(self):
        return C.byref(self.c)


def dllava_predict_workspace(M: int, B: int, n_blocks: int) -> int:
    return _lib.dllava_predict_workspace(M, B, n_blocks)


def dllava_predict(x, ldx, M, B, seq_off, vis_start, vis_len, p: Predictor, dtype, logits, workspace, stream=None):
    ws, nbytes = _ws(workspace)
    _check(_lib.dllava_predict(_p(x), ldx, M, B, _p(seq_off), _p(vis_start), _p(vis_len), p.ref, dtype, _p(logits),
                               ws, nbytes, _stream(stream)))


def dllava_compact(B, seq_off, kept_idx, out_off, sumN, hidden, hidden_out, d, Q, Q_out, K, V, cache, err_flag, dtype,
                   stream=None):
    _check(_lib.dllava_compact(B, _p(seq_off), _p(kept_idx), _p(out_off), sumN, _p(hidden), _p(hidden_out), d, _p(Q),
                               _p(Q_out), _p(K), _p(V), cache.ref if cache is not None else None, _p(err_flag), dtype,
                               _stream(stream)))


def dllava_masked_attn_workspace(rows: int, B: int) -> int:
    return _lib.dllava_masked_attn_workspace(rows, B)


def dllava_masked_attn(Q, K, V, B, off, rows, H, Dh, scale, keep_mask, O, dtype, workspace, stream=None):
    ws, nbytes = _ws(workspace)
    _check(_lib.dllava_masked_attn(_p(Q), _p(K), _p(V), B, _p(off), rows, H, Dh, scale, _p(keep_mask), _p(O), dtype,
                                   ws, nbytes, _stream(stream)))


def dllava_linear(x, ldx, M, K, W, bias, N, act, residual, y, ldy, dtype, stream=None):
    _check(_lib.dllava_linear(_p(x), ldx, M, K, _p(W), _p(bias), N, act, _p(residual), _p(y), ldy, dtype, _stream(stream)))


def dllava_layer_norm(z, M, gamma, beta, y, dtype, stream=None):
    _check(_lib.dllava_layer_norm(_p(z), M, _p(gamma), _p(beta), _p(y), dtype, _stream(stream)))


def dllava_linear_few_workspace(N: int, K: int) -> int:
    return _lib.dllava_linear_few_workspace(N, K)


def dllava_linear_few(x, ldx, M, K, W, bias, N, act, residual, y, ldy, dtype, workspace, stream=None):
    ws, nbytes = _ws(workspace)
    _check(_lib.dllava_linear_few(_p(x), ldx, M, K, _p(W), _p(bias), N, act, _p(residual), _p(y), ldy, dtype, ws, nbytes,
                                  _stream(stream)))


def dllava_decode_proj_workspace(N_total: int, K: int) -> int:
    return _lib.dllava_decode_proj_workspace(N_total, K)


def dllava_qkv_few(x, ldx, M, d, Wq, Wk, Wv, H, Dh, pos, rope_base, q, k, v, dtype, workspace, stream=None):
    ws, nbytes = _ws(workspace)
    _check(_lib.dllava_qkv_few(_p(x), ldx, M, d, _p(Wq), _p(Wk), _p(Wv), H, Dh, _p(pos), rope_base, _p(q), _p(k), _p(v),
                               dtype, ws, nbytes, _stream(stream)))


def dllava_gated_few(x, ldx, M, d, Wg, Wu, F, y, ldy, dtype, workspace, stream=None):
    ws, nbytes = _ws(workspace)
    _check(_lib.dllava_gated_few(_p(x), ldx, M, d, _p(Wg), _p(Wu), F, _p(y), ldy, dtype, ws, nbytes, _stream(stream)))


def dllava_rope(x, pos, rows, H, Dh, rope_base, dtype, stream=None):
    _check(_lib.dllava_rope(_p(x), _p(pos), rows, H, Dh, rope_base, dtype, _stream(stream)))


def dllava_rms_norm(x, ldx, M, d, weight, eps, y, ldy, dtype, stream=None):
    _check(_lib.dllava_rms_norm(_p(x), ldx, M, d, _p(weight), eps, _p(y), ldy, dtype, _stream(stream)))


def dllava_span_attn(Q, K, V, B, off, rows, H, Dh, scale, O, dtype, stream=None):
    _check(_lib.dllava_span_attn(_p(Q), _p(K), _p(V), B, _p(off), rows, H, Dh, scale, _p(O), dtype, _stream(stream)))


def dllava_version() -> int:
    return _lib.dllava_version()


def dllava_set_launch_override(knob: int, value: int) -> None:
    _check(_lib.dllava_set_launch_override(knob, value))


def dllava_score_workspace(M: int, d: int, dh: int, dtype: int) -> int:
    return _lib.dllava_score_workspace(M, d, dh, dtype)


def dllava_select_compact_workspace(B: int, sumN: int) -> int:
    return _lib.dllava_select_compact_workspace(B, sumN)


def dllava_decode_workspace(B: int, H: int, Dh: int, max_pages_per_seq: int) -> int:
    return _lib.dllava_decode_workspace(B, H, Dh, max_pages_per_seq)


def dllava_score(x, ldx, M, B, seq_off, vis_start, vis_len, d, dh, W1, b1, W2, b2, dtype, logits,
                 workspace, stream=None) -> None:
    wp, wb = _ws(workspace)
    _check(_lib.dllava_score(_p(x), ldx, M, B, _p(seq_off), _p(vis_start), _p(vis_len), d, dh, _p(W1), _p(b1),
                             _p(W2), _p(b2), dtype, _p(logits), wp, wb, _stream(stream)))


def dllava_select_compact(logits, B, seq_off, vis_start, vis_len, sumN, mode, keep_ratio, threshold,
                          hidden, hidden_out, d, Q, Q_out, K, V, cache: Optional[KVCache],
                          keep_mask, kept_idx, out_off, err_flag, dtype, workspace, stream=None) -> None:
    wp, wb = _ws(workspace)
    _check(_lib.dllava_select_compact(_p(logits), B, _p(seq_off), _p(vis_start), _p(vis_len), sumN, mode,
                                      keep_ratio, threshold, _p(hidden), _p(hidden_out), d, _p(Q), _p(Q_out),
                                      _p(K), _p(V), cache.ref if cache is not None else None, _p(keep_mask),
                                      _p(kept_idx), _p(out_off), _p(err_flag), dtype, wp, wb, _stream(stream)))


def dllava_prefill_attn(Q, K, V, cache: Optional[KVCache], B, off, rows, H, Dh, scale, O, dtype,
                        stream=None) -> None:
    _check(_lib.dllava_prefill_attn(_p(Q), _p(K), _p(V), cache.ref if cache is not None else None, B, _p(off),
                                    rows, H, Dh, scale, _p(O), dtype, _stream(stream)))


def dllava_decode_step_workspace(B: int, H: int, Dh: int, max_pages_per_seq: int, d: int, dh: int, dtype: int) -> int:
    return int(_lib.dllava_decode_step_workspace(B, H, Dh, max_pages_per_seq, d, dh, dtype))


def dllava_decode_step(x, ldx, d, dh, W1, b1, W2, b2, q, k_new, v_new, k_prev, v_prev, logits_prev,
                       keep_prev_override, B, threshold, cache: KVCache, scale, o, logits, keep_prev_out, err_flag,
                       workspace, stream=None) -> None:
    wp, wb = _ws(workspace)
    _check(_lib.dllava_decode_step(_p(x), ldx, d, dh, _p(W1), _p(b1), _p(W2), _p(b2), _p(q), _p(k_new), _p(v_new),
                                   _p(k_prev), _p(v_prev), _p(logits_prev), _p(keep_prev_override), B, threshold,
                                   cache.ref, scale, _p(o), _p(logits), _p(keep_prev_out), _p(err_flag), wp, wb,
                                   _stream(stream)))


def dllava_decode_commit(k_prev, v_prev, logits_prev, keep_prev_override, B, threshold, cache: KVCache, keep_out,
                         err_flag, stream=None) -> None:
    _check(_lib.dllava_decode_commit(_p(k_prev), _p(v_prev), _p(logits_prev), _p(keep_prev_override), B, threshold,
                                     cache.ref, _p(keep_out), _p(err_flag), _stream(stream)))


def dllava_qkv_project(x, ldx, rows, d, B, off, pos, Wq, Wk, Wv, rope_base, Q_out, cache: KVCache, err_flag, dtype,
                       stream=None) -> None:
    _check(_lib.dllava_qkv_project(_p(x), ldx, rows, d, B, _p(off), _p(pos), _p(Wq), _p(Wk), _p(Wv), rope_base,
                                   _p(Q_out), cache.ref, _p(err_flag), dtype, _stream(stream)))


def dllava_decode_attn_append(q, k_new, v_new, B, logits, threshold, keep_override, cache: KVCache, scale,
                              o, keep_out, err_flag, workspace, stream=None) -> None:
    wp, wb = _ws(workspace)
    _check(_lib.dllava_decode_attn_append(_p(q), _p(k_new), _p(v_new), B, _p(logits), threshold,
                                          _p(keep_override), cache.ref, scale, _p(o), _p(keep_out),
                                          _p(err_flag), wp, wb, _stream(stream)))



def dllava_decode_attn_append_static(q, k_new, v_new, B, logits, threshold, keep_override, cache: KVCache, scale,
                                     o, keep_out, err_flag, stream=None) -> None:
    _check(_lib.dllava_decode_attn_append_static(_p(q), _p(k_new), _p(v_new), B, _p(logits), threshold,
                                                 _p(keep_override), cache.ref, scale, _p(o), _p(keep_out),
                                                 _p(err_flag), _stream(stream)))


def _bind_native() -> None:
    torch_here = f"{torch.__version__} {torch.version.git_version}"
    try:
        from . import _calls
        if getattr(_calls, "torch_version", None) != torch_here:  # its layouts are that torch's
            raise ImportError(f"_calls was built for torch {getattr(_calls, 'torch_version', '(not named)')}, this is {torch_here}")
    except ImportError as e:
        warnings.warn(f"calls take their arguments through ctypes, a few microseconds longer each: {e} "
                      "(`python -m paper_2412_00876_amd.build` builds the native forms)", RuntimeWarning, stacklevel=2)
        return
    _calls.init(KVCache, Predictor, _check, torch.cuda.current_device, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
    for name in EXPORTS:
        python = globals().get(name)
        if python is None:
            continue
        code = python.__code__
        names = code.co_varnames[:code.co_argcount]
        if names and names[-1] == "stream":
            function = getattr(_lib, name)
            native = _calls.bind(name, python, names, function, C.cast(function, C.c_void_p).value)
            globals()[name] = functools.update_wrapper(native, python)


_bind_native()
