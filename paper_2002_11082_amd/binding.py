"""Binding of libogq's C ABI (include/ogq.h): ctypes for the raw calls and the size queries, the extension module
_marshal (csrc/torch_marshal.cpp) for the two calls on tensors.  Argument marshalling only: every step of the path runs in
the HIP kernels.  There is no CPU fallback: a missing library is an error."""
from __future__ import annotations

import ctypes
import os

_PKG = os.path.dirname(os.path.abspath(__file__))
# OGQ_LIBRARY names another build of the same C ABI (e.g. a host build with sanitizers for the argument checks).
LIB_PATH = os.environ.get("OGQ_LIBRARY") or os.path.join(_PKG, "libogq.so")

BINGRAD_B = 0
ORQ = 1
BINGRAD_PB = 2
ORQ_PAPER = 3
SCALED_SIGN = 4
EVEN = 5
LINEAR = 6
MAX_WORKERS = 64
PROBE_SINK_FLOATS = 8192


class Params(ctypes.Structure):
    """ogq_params_t"""
    _fields_ = [
        ("bucket_size", ctypes.c_uint32),
        ("bits", ctypes.c_uint32),
        ("scheme", ctypes.c_uint32),
        ("level_iters", ctypes.c_uint32),
        ("seed", ctypes.c_uint64),
        ("index_offset", ctypes.c_uint64),
        ("clip_factor", ctypes.c_float),
        ("reserved", ctypes.c_uint32),
    ]


class OgqError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"libogq status {status}: {text}")
        self.status = status


_lib = None


def lib() -> ctypes.CDLL:
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(
                f"{LIB_PATH} is missing: build it with `python -m paper_2002_11082_amd.build` "
                "(there is no CPU fallback)")
        L = ctypes.CDLL(LIB_PATH)
        sz, vp, u32 = ctypes.c_size_t, ctypes.c_void_p, ctypes.c_uint32
        pp = ctypes.POINTER(Params)
        L.ogq_levels_per_bucket.argtypes = [pp]
        L.ogq_levels_per_bucket.restype = sz
        for name in ("ogq_num_buckets", "ogq_levels_count", "ogq_codes_bytes"):
            f = getattr(L, name)
            f.argtypes = [sz, pp]
            f.restype = sz
        L.ogq_quantize.argtypes = [vp, sz, pp, vp, vp, vp]
        L.ogq_quantize.restype = ctypes.c_int
        L.ogq_dequantize_average.argtypes = [vp, vp, u32, sz, pp, vp, vp]
        L.ogq_dequantize_average.restype = ctypes.c_int
        L.ogq_probe_read.argtypes = [vp, sz, vp, vp]
        L.ogq_probe_read.restype = ctypes.c_int
        L.ogq_probe_copy.argtypes = [vp, vp, sz, vp]
        L.ogq_probe_copy.restype = ctypes.c_int
        L.ogq_strerror.argtypes = [ctypes.c_int]
        L.ogq_strerror.restype = ctypes.c_char_p
        L.ogq_last_hip_error.argtypes = []
        L.ogq_last_hip_error.restype = ctypes.c_int
        _lib = L
    return _lib


def make_params(bucket_size: int, bits: int, scheme: int, level_iters: int = 0, seed: int = 0,
                index_offset: int = 0, clip_factor: float = 0.0) -> Params:
    return Params(bucket_size, bits, scheme, level_iters, seed, index_offset, clip_factor, 0)


def ogq_strerror(status: int) -> str:
    return lib().ogq_strerror(status).decode()


def _check(status: int) -> None:
    if status != 0:
        raise OgqError(status, ogq_strerror(status))


def ogq_levels_per_bucket(params: Params) -> int:
    return lib().ogq_levels_per_bucket(ctypes.byref(params))


def ogq_num_buckets(n: int, params: Params) -> int:
    return lib().ogq_num_buckets(n, ctypes.byref(params))


def ogq_levels_count(n: int, params: Params) -> int:
    return lib().ogq_levels_count(n, ctypes.byref(params))


def ogq_codes_bytes(n: int, params: Params) -> int:
    return lib().ogq_codes_bytes(n, ctypes.byref(params))


def ogq_quantize_raw(d_grad: int, n: int, params: Params, d_levels: int, d_codes: int, stream: int = 0) -> int:
    """Raw call: device addresses as integers; returns the status code."""
    return lib().ogq_quantize(d_grad, n, ctypes.byref(params), d_levels, d_codes, stream)


def ogq_dequantize_average_raw(d_codes, d_levels, n: int, params: Params, d_out: int, stream: int = 0) -> int:
    """Raw call: d_codes / d_levels are sequences of device addresses; returns the status code."""
    W = len(d_codes)
    cp = (ctypes.c_void_p * max(W, 1))(*d_codes)
    lp = (ctypes.c_void_p * max(W, 1))(*d_levels)
    return lib().ogq_dequantize_average(ctypes.addressof(cp), ctypes.addressof(lp), W, n, ctypes.byref(params),
                                        d_out, stream)


def _stream_of(t) -> int:
    import torch
    return torch.cuda.current_stream(t.device).cuda_stream


_marshal = None


def _load_marshal():
    """The extension module that takes tensors, bound to this process's library."""
    global _marshal
    import torch  # first: the module links against torch's libraries
    try:
        from . import _marshal as module
    except ImportError as e:
        raise ImportError(f"the extension module _marshal cannot be loaded ({e}): build it with "
                          "`python -m paper_2002_11082_amd.build`") from e
    L = lib()
    addresses = [ctypes.cast(f, ctypes.c_void_p).value
                 for f in (L.ogq_quantize, L.ogq_dequantize_average, L.ogq_levels_count, L.ogq_codes_bytes)]
    module.bind(*addresses, torch._C._cuda_getCurrentRawStream, _check, Params)
    _marshal = module
    return module


def ogq_quantize(grad, params: Params, levels=None, codes=None):
    """grad: 1-D contiguous float32 CUDA tensor.  Returns (levels float32[levels_count],
    codes int64[codes_bytes/8]) on the same device, enqueued on torch's current stream."""
    return (_marshal or _load_marshal()).quantize(grad, params, levels, codes)


def ogq_dequantize_average(codes_list, levels_list, n: int, params: Params, out=None):
    """codes_list / levels_list: one CUDA tensor per worker as returned by ogq_quantize.
    Returns float32[n]."""
    return (_marshal or _load_marshal()).dequantize_average(codes_list, levels_list, n, params, out)


def ogq_probe_read(src, sink=None):
    import torch
    if sink is None:
        sink = torch.empty(PROBE_SINK_FLOATS, dtype=torch.float32, device=src.device)
    _check(lib().ogq_probe_read(src.data_ptr(), src.numel(), sink.data_ptr(), _stream_of(src)))
    return sink


def ogq_probe_copy(src, dst):
    _check(lib().ogq_probe_copy(src.data_ptr(), dst.data_ptr(), src.numel(), _stream_of(src)))
    return dst
