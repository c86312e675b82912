"""Binding of libmosaicattn.so: same names as the C ABI, argument marshalling only.

Tensors are torch tensors used purely as device buffers (data_ptr, shape, stride); every step of
the path runs inside the HIP library.  Importing this module raises if the library is not built:
there is no CPU or PyTorch fallback.  The calls that a step makes many times are marshalled by native code
(csrc/marshal.cpp), the others by ctypes.
"""
from __future__ import annotations

import copyreg
import ctypes
import importlib.machinery
import importlib.util
import os
from ctypes import c_char_p, c_float, c_int, c_int64, c_size_t, c_void_p

import torch

_LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "lib", "libmosaicattn.so")
_MARSHAL_PATH = os.path.join(os.path.dirname(_LIB_PATH), "_mosaic_marshal.so")
_HOW_TO_BUILD = "Run `python -c 'import __graft_entry__ as g; g.build()'`."
for _path in (_LIB_PATH, _MARSHAL_PATH):
    if not os.path.exists(_path):
        raise ImportError("%s is not built (%s). %s" % (os.path.basename(_path), _path, _HOW_TO_BUILD))
_lib = ctypes.CDLL(_LIB_PATH)

MB_OK, MB_ERR_INVALID_ARG, MB_ERR_UNSUPPORTED, MB_ERR_WORKSPACE, MB_ERR_HIP = range(5)
MB_F32, MB_BF16 = 0, 1

EXPORTS = ("mb_last_error", "mb_version", "mb_alibi_slopes", "mb_unpad_index", "mb_read_meta", "mb_unpad",
           "mb_pad", "mb_zero_padding", "mb_alibi_attn_fwd", "mb_alibi_attn_fwd_workspace_bytes",
           "mb_alibi_attn_bwd_workspace_bytes",
           "mb_alibi_attn_bwd", "mb_add_layernorm_fwd", "mb_add_layernorm_bwd_workspace_bytes",
           "mb_add_layernorm_bwd", "mb_geglu_fwd", "mb_geglu_bwd_workspace_bytes", "mb_geglu_bwd", "mb_linear_fwd", "mb_gelu_gate", "mb_probe_ceiling",
           "mb_alibi_attn_bwd_static", "mb_device_status", "mb_attn_plan_bytes", "mb_attn_plan", "mb_probe_bwd_traffic")

_lib.mb_last_error.restype = c_char_p
_lib.mb_last_error.argtypes = []
_lib.mb_version.restype = c_int
_lib.mb_version.argtypes = []
_lib.mb_alibi_slopes.restype = c_int
_lib.mb_alibi_slopes.argtypes = [c_int, c_void_p]
_lib.mb_unpad_index.restype = c_int
_lib.mb_unpad_index.argtypes = [c_void_p, c_int, c_int, c_void_p, c_void_p, c_void_p, c_void_p, c_void_p]
_lib.mb_read_meta.restype = c_int
_lib.mb_read_meta.argtypes = [c_void_p, c_void_p, c_void_p]
_lib.mb_unpad.restype = c_int
_lib.mb_unpad.argtypes = [c_void_p, c_void_p, c_int, c_void_p, c_int, c_int, c_void_p, c_void_p]
_lib.mb_pad.restype = c_int
_lib.mb_pad.argtypes = [c_void_p, c_void_p, c_int, c_void_p, c_int, c_int, c_int, c_int, c_void_p, c_void_p]
_lib.mb_zero_padding.restype = c_int
_lib.mb_zero_padding.argtypes = [c_void_p, c_int, c_void_p, c_int, c_int, c_int, c_int, c_void_p, c_void_p]
_lib.mb_alibi_attn_fwd.restype = c_int
_lib.mb_alibi_attn_fwd.argtypes = [c_void_p, c_void_p, c_void_p, c_int64, c_int64, c_int64, c_void_p, c_int, c_int,
                                   c_int, c_int, c_int, c_void_p, c_float, c_int, c_void_p, c_int64, c_void_p,
                                   c_void_p, c_size_t, c_void_p, c_void_p, c_void_p, c_void_p]
_lib.mb_attn_plan_bytes.restype = c_size_t
_lib.mb_attn_plan_bytes.argtypes = [c_int, c_int, c_int]
_lib.mb_attn_plan.restype = c_int
_lib.mb_attn_plan.argtypes = [c_void_p, c_void_p, c_int, c_int, c_int, c_void_p, c_size_t, c_void_p]
_lib.mb_alibi_attn_fwd_workspace_bytes.restype = c_size_t
_lib.mb_alibi_attn_fwd_workspace_bytes.argtypes = [c_int, c_int, c_int, c_int, c_int, c_int]
_lib.mb_alibi_attn_bwd_workspace_bytes.restype = c_size_t
_lib.mb_alibi_attn_bwd_workspace_bytes.argtypes = [c_int, c_int, c_int, c_int, c_int, c_int]
_lib.mb_alibi_attn_bwd.restype = c_int
_lib.mb_alibi_attn_bwd.argtypes = ([c_void_p] * 6 + [c_int64] * 5 + [c_void_p] + [c_int] * 5 + [c_void_p, c_float, c_int]
                                   + [c_void_p] * 3 + [c_int64] * 3
                                   + [c_void_p, c_size_t, c_void_p, c_void_p, c_void_p, c_void_p])
_lib.mb_alibi_attn_bwd_static.restype = c_int
_lib.mb_alibi_attn_bwd_static.argtypes = ([c_void_p] * 6 + [c_int64] * 5 + [c_void_p] + [c_int] * 5
                                          + [c_void_p, c_float, c_int] + [c_void_p] * 3 + [c_int64] * 3
                                          + [c_void_p, c_void_p, c_void_p, c_void_p])
_lib.mb_device_status.restype = c_int
_lib.mb_device_status.argtypes = [c_void_p]
MB_STATIC_SCRATCH_BYTES = 16 << 20

_lib.mb_add_layernorm_fwd.restype = c_int
_lib.mb_add_layernorm_fwd.argtypes = [c_void_p, c_void_p, c_void_p, c_void_p, c_int, c_void_p, c_int, c_float, c_int,
                                      c_void_p, c_void_p, c_void_p, c_void_p, c_void_p, c_void_p]
_lib.mb_add_layernorm_bwd_workspace_bytes.restype = c_size_t
_lib.mb_add_layernorm_bwd_workspace_bytes.argtypes = [c_int]
_lib.mb_add_layernorm_bwd.restype = c_int
_lib.mb_add_layernorm_bwd.argtypes = [c_void_p, c_void_p, c_void_p, c_void_p, c_void_p, c_int, c_void_p, c_int, c_int,
                                      c_void_p, c_void_p, c_void_p, c_void_p, c_size_t, c_void_p, c_void_p]
_lib.mb_geglu_bwd_workspace_bytes.restype = c_size_t
_lib.mb_geglu_bwd_workspace_bytes.argtypes = [c_int, c_int, c_int, c_int]
_lib.mb_geglu_bwd.restype = c_int
_lib.mb_geglu_bwd.argtypes = [c_void_p, c_void_p, c_void_p, c_void_p, c_void_p, c_void_p, c_int, c_void_p, c_int, c_int, c_int,
                              c_void_p, c_void_p, c_void_p, c_void_p, c_size_t, c_void_p]
_lib.mb_probe_bwd_traffic.restype = c_int
_lib.mb_probe_bwd_traffic.argtypes = [c_void_p, c_void_p, c_void_p, c_void_p, c_void_p, c_int, c_int, c_void_p]
_lib.mb_probe_ceiling.restype = c_int
_lib.mb_probe_ceiling.argtypes = [c_int, c_int, c_void_p, c_void_p, c_void_p]
_lib.mb_linear_fwd.restype = c_int
_lib.mb_linear_fwd.argtypes = [c_void_p, c_void_p, c_int, c_void_p, c_int, c_int, c_int, c_void_p, c_void_p]
_lib.mb_gelu_gate.restype = c_int
_lib.mb_gelu_gate.argtypes = [c_void_p, c_void_p, c_int64, c_int, c_void_p, c_int, c_int, c_void_p, c_void_p]
_lib.mb_geglu_fwd.restype = c_int
_lib.mb_geglu_fwd.argtypes = [c_void_p, c_void_p, c_void_p, c_int, c_void_p, c_int, c_int, c_int, c_void_p, c_void_p,
                              c_void_p]


class MosaicAttnError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__("libmosaicattn status %d: %s" % (status, message))
        self.status = status


def raw():
    """The ctypes library handle, for tests of the C ABI itself."""
    return _lib


def _check(status: int) -> None:
    if status != MB_OK:
        raise MosaicAttnError(status, _lib.mb_last_error().decode())


_DTYPE_CODES = {torch.float32: MB_F32, torch.bfloat16: MB_BF16}
_current_device = torch.cuda.current_device
# (torch.cuda.current_stream() makes a Stream object on every call.  A torch without a GPU backend has no such function:
# this module can be imported there all the same, for the host-side calls.)
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _ptr(t) -> int | None:
    return None if t is None else t.data_ptr()


def _stream() -> int:
    if _raw_stream is None:
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(_current_device())


def _dtype_code(t: torch.Tensor) -> int:
    code = _DTYPE_CODES.get(t.dtype)
    if code is None:
        raise TypeError("unsupported dtype %s" % t.dtype)
    return code


def _row_stride(t: torch.Tensor) -> int:
    """[T, H, D] view with contiguous (H, D): returns the token stride in elements."""
    shape, strides = t.shape, t.stride()
    assert len(strides) == 3 and strides[2] == 1 and strides[1] == shape[2], "need [T, H, D] with dense (H, D)"
    return strides[0] if shape[0] > 1 else max(strides[0], shape[1] * shape[2])


def _load_calls():
    """The native calls of this module (its own object: another import of the binding has its own error class)."""
    loader = importlib.machinery.ExtensionFileLoader("_mosaic_marshal", _MARSHAL_PATH)
    try:
        native = importlib.util.module_from_spec(importlib.util.spec_from_loader("_mosaic_marshal", loader))
        loader.exec_module(native)
        if not torch.__version__.startswith(native.torch_version):   # may load all the same, with other layouts
            raise ImportError("built for torch " + native.torch_version)
    except ImportError as e:   # it is compiled against the headers of one Python and one torch
        raise ImportError("%s does not load with torch %s; it was built for another one, or not whole. %s"
                          % (_MARSHAL_PATH, torch.__version__, _HOW_TO_BUILD)) from e
    addresses = {name: ctypes.cast(getattr(_lib, name), c_void_p).value for name in EXPORTS}
    return native.Calls(addresses, MosaicAttnError, getattr(torch._C, "_cuda_getDevice", _current_device), _raw_stream,
                        _stream)


# Host time of a whole layer step of 8 x 128 positions, eight calls (33 us of kernels): 60 us with these calls marshalled in
# Python; see csrc/marshal.cpp.
_calls = _load_calls()


def _calls_of_this_module():
    return _calls


copyreg.pickle(type(_calls), lambda _: (_calls_of_this_module, ()))   # its methods pickle by name, as functions do

mb_unpad_index = _calls.mb_unpad_index
mb_unpad = _calls.mb_unpad
mb_pad = _calls.mb_pad
mb_zero_padding = _calls.mb_zero_padding
mb_alibi_attn_fwd = _calls.mb_alibi_attn_fwd
mb_alibi_attn_bwd = _calls.mb_alibi_attn_bwd
mb_add_layernorm_fwd = _calls.mb_add_layernorm_fwd
mb_add_layernorm_bwd = _calls.mb_add_layernorm_bwd
mb_geglu_fwd = _calls.mb_geglu_fwd
mb_geglu_bwd = _calls.mb_geglu_bwd
mb_linear_fwd = _calls.mb_linear_fwd


def mb_version() -> int:
    return _lib.mb_version()


def mb_last_error() -> str:
    return _lib.mb_last_error().decode()


def mb_alibi_slopes(H: int) -> torch.Tensor:
    """Host tensor [H] float32 of the head slopes."""
    out = torch.empty(max(H, 0), dtype=torch.float32)
    _check(_lib.mb_alibi_slopes(H, out.data_ptr() if H > 0 else None))
    return out


def mb_read_meta(meta: torch.Tensor):
    host = (ctypes.c_int32 * 2)()
    _check(_lib.mb_read_meta(_ptr(meta), ctypes.addressof(host), _stream()))
    return int(host[0]), int(host[1])


def mb_attn_plan_bytes(B: int, max_seqlen: int, H: int) -> int:
    return int(_lib.mb_attn_plan_bytes(B, max_seqlen, H))


def mb_attn_plan(cu_seqlens, max_seqlen: int, H: int, key_lens=None, plan=None):
    """Builds the work plan of the any-length attention kernels once for a batch; returns the plan buffer."""
    B = cu_seqlens.numel() - 1
    need = mb_attn_plan_bytes(B, max_seqlen, H)
    if plan is None:
        plan = torch.empty(max(need, 16), dtype=torch.uint8, device=cu_seqlens.device)
    _check(_lib.mb_attn_plan(_ptr(cu_seqlens), _ptr(key_lens), B, max_seqlen, H, _ptr(plan), plan.numel(), _stream()))
    return plan


def mb_alibi_attn_fwd_workspace_bytes(B, T, max_seqlen, H, D, dtype_code) -> int:
    return int(_lib.mb_alibi_attn_fwd_workspace_bytes(B, T, max_seqlen, H, D, dtype_code))


def mb_alibi_attn_bwd_workspace_bytes(B, T, max_seqlen, H, D, dtype_code) -> int:
    return int(_lib.mb_alibi_attn_bwd_workspace_bytes(B, T, max_seqlen, H, D, dtype_code))


def mb_alibi_attn_bwd_static(dout, q, k, v, o, lse, cu_seqlens, max_seqlen: int, slopes, softmax_scale: float,
                             dq, dk, dv, token_rows=None, T=None, key_lens=None, plan=None):
    """mb_alibi_attn_bwd on the library's static scratch array.  This wrapper allocates nothing either:
    the outputs dq, dk, dv must be given."""
    R, H, D = q.shape
    T = R if T is None else T
    B = cu_seqlens.numel() - 1
    _check(_lib.mb_alibi_attn_bwd_static(_ptr(dout), _ptr(q), _ptr(k), _ptr(v), _ptr(o), _ptr(lse), _row_stride(dout),
                                         _row_stride(q), _row_stride(k), _row_stride(v), _row_stride(o),
                                         _ptr(cu_seqlens), B, T, max_seqlen, H, D, _ptr(slopes), float(softmax_scale),
                                         _dtype_code(q), _ptr(dq), _ptr(dk), _ptr(dv), _row_stride(dq),
                                         _row_stride(dk), _row_stride(dv), _ptr(key_lens), _ptr(token_rows), _ptr(plan),
                                         _stream()))
    return dq, dk, dv


def mb_device_status() -> None:
    """Raises MosaicAttnError(MB_ERR_INVALID_ARG) if an attention call since the last check met a sequence
    longer than its max_seqlen; clears the device's sticky word.  Synchronises the current stream."""
    _check(_lib.mb_device_status(_stream()))


def mb_add_layernorm_bwd_workspace_bytes(W: int) -> int:
    return int(_lib.mb_add_layernorm_bwd_workspace_bytes(W))


def mb_gelu_gate(h, gate, T_cap=None, meta=None, act=None):
    """act = GeLU(h) * gate; h and gate are [rows, inter] views with the same row stride (two buffers, or
    the halves of one [rows, 2*inter] buffer)."""
    assert h.dim() == 2 and h.shape == gate.shape and h.stride(1) == 1 and gate.stride(1) == 1
    assert h.stride(0) == gate.stride(0)
    rows, inter = h.shape
    T_cap = rows if T_cap is None else T_cap
    act = torch.empty((rows, inter), dtype=h.dtype, device=h.device) if act is None else act
    _check(_lib.mb_gelu_gate(_ptr(h), _ptr(gate), h.stride(0), T_cap, _ptr(meta), inter, _dtype_code(h), _ptr(act),
                             _stream()))
    return act


def mb_probe_ceiling(kind: int, iters: int, out) -> float:
    """Enqueues one probe launch (0: bf16 MFMA, 1: fp32 FMA, 2: fp32 exp); returns its work (flops or exps)."""
    work = ctypes.c_double(0.0)
    _check(_lib.mb_probe_ceiling(kind, iters, _ptr(out), ctypes.byref(work), _stream()))
    return work.value


def mb_probe_bwd_traffic(qkv, dout, o, dqkv, cu_seqlens) -> None:
    """Enqueues the traffic-only twin of the single-tile backward: qkv [T, 3, H, 64], dout / o [T, H, 64] read,
    dqkv [T, 3, H, 64] overwritten with meaningless values."""
    H = dout.shape[1]
    assert qkv.is_contiguous() and dout.is_contiguous() and o.is_contiguous() and dqkv.is_contiguous()
    _check(_lib.mb_probe_bwd_traffic(_ptr(qkv), _ptr(dout), _ptr(o), _ptr(dqkv), _ptr(cu_seqlens),
                                     cu_seqlens.numel() - 1, H, _stream()))


def mb_geglu_bwd_workspace_bytes(T_cap: int, hidden: int, inter: int, dtype_code: int = MB_BF16) -> int:
    return int(_lib.mb_geglu_bwd_workspace_bytes(T_cap, hidden, inter, dtype_code))
