"""Binding of libhago.so: same names as the C ABI, argument marshalling only.

Tensors are torch tensors on the GPU; the binding passes their device pointers
and the current torch stream to the library and allocates the output tensor.
The operators are marshalled by a native module (csrc/native.cpp), everything
around them by ctypes.  There is no CPU fallback: if the library is missing,
loading fails.
"""
from __future__ import annotations

import ctypes as C
import os

U8, I8, I16, I32, F32, I24 = 0, 1, 2, 3, 4, 5   # I24: accumulator / simulated type only
NCHW, NHWC = 0, 1
STRICT_ACC16 = 1
WS_WEIGHTS_READY = 2
STATIC_SCRATCH_BYTES = 64 << 20   # HAGO_STATIC_SCRATCH_BYTES
HOOK_GEMM_PATH, HOOK_STREAM_TILE, HOOK_GENERAL_TILE = 0, 1, 2   # hago_set_test_hook keys
ROUND_UPWARD, ROUND_HALF_AWAY = 0, 1   # hago_rounding

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libhago.so")
_NATIVE_PATH = os.path.join(_HERE, "_native.so")

EXPORTS = ("hago_simquant", "hago_simquant_batched", "hago_absmax", "hago_simquant_wrap", "hago_quantize", "hago_dequantize", "hago_simquant_codes", "hago_qdense", "hago_qconv2d", "hago_qconv2d_ws", "hago_qconv2d_workspace_bytes", "hago_qconv2d_static", "hago_requantize",
           "hago_status_string", "hago_bit_range", "hago_set_test_hook", "hago_probe_mfma_i8", "hago_probe_copy")


class _QType(C.Structure):
    _fields_ = [("dtype", C.c_int32), ("bits", C.c_int32), ("is_signed", C.c_int32),
                ("zero_point", C.c_int32)]


class _Requant(C.Structure):
    _fields_ = [("multiplier", C.c_void_p), ("shift", C.c_void_p), ("per_channel", C.c_int32),
                ("out", _QType), ("clip_lo", C.c_int32), ("clip_hi", C.c_int32), ("rounding", C.c_int32)]


class HagoError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__(f"libhago: {msg} (status {code})")
        self.code = code


def library_path() -> str:
    return _LIB_PATH


_lib = None
_native = None


def lib():
    """Load libhago.so (built by paper_2103_14949_amd/build.py); raises if absent."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise FileNotFoundError(
                f"{_LIB_PATH} is missing: build it with `python -m paper_2103_14949_amd.build` "
                "(there is no fallback path)")
        L = C.CDLL(_LIB_PATH)
        i32, i64, u32, vp = C.c_int32, C.c_int64, C.c_uint32, C.c_void_p
        L.hago_status_string.restype = C.c_char_p
        L.hago_status_string.argtypes = [i32]
        L.hago_simquant.restype = i32
        L.hago_simquant.argtypes = [vp, vp, i64, i64, i64, vp, vp, i32, _QType, i32, i32, vp]
        L.hago_simquant_wrap.restype = i32
        L.hago_simquant_wrap.argtypes = L.hago_simquant.argtypes
        L.hago_simquant_batched.restype = i32
        L.hago_simquant_batched.argtypes = [vp, vp, i64, i64, i64, i32, vp, vp, i32, _QType, vp, vp, vp]
        L.hago_quantize.restype = i32
        L.hago_quantize.argtypes = [vp, vp, i64, i64, i64, vp, vp, i32, _QType, i32, i32, vp]
        L.hago_simquant_codes.restype = i32
        L.hago_simquant_codes.argtypes = [vp, vp, vp, i64, i64, i64, vp, vp, i32, _QType, i32, i32, vp]
        L.hago_dequantize.restype = i32
        L.hago_dequantize.argtypes = [vp, _QType, vp, i64, i64, i64, vp, vp, i32, vp]
        L.hago_absmax.restype = i32
        L.hago_absmax.argtypes = [vp, i64, i64, i64, i32, vp, vp]
        L.hago_requantize.restype = i32
        L.hago_requantize.argtypes = [vp, i32, i64, i64, i64, C.POINTER(_Requant), vp, vp]
        L.hago_qdense.restype = i32
        L.hago_qdense.argtypes = [vp, _QType, vp, _QType, vp, i64, i64, i64, i32,
                                  C.POINTER(_Requant), vp, u32, vp]
        L.hago_qconv2d.restype = i32
        L.hago_qconv2d.argtypes = [vp, _QType, vp, _QType, vp, i32, i64, i64, i64, i64, i64,
                                   i32, i32, i32, i32, i32, i32, i32, i32,
                                   C.POINTER(_Requant), vp, u32, vp]
        L.hago_qconv2d_static.restype = i32
        L.hago_qconv2d_static.argtypes = L.hago_qconv2d.argtypes
        L.hago_qconv2d_ws.restype = i32
        L.hago_qconv2d_ws.argtypes = [vp, _QType, vp, _QType, vp, i32, i64, i64, i64, i64, i64,
                                      i32, i32, i32, i32, i32, i32, i32, i32,
                                      C.POINTER(_Requant), vp, vp, i64, u32, vp]
        L.hago_qconv2d_workspace_bytes.restype = i64
        L.hago_qconv2d_workspace_bytes.argtypes = [i32, i64, i64, i64, i64, i64, i32, i32, i32, i32, i32, i32, i32]
        L.hago_bit_range.restype = i32
        L.hago_bit_range.argtypes = [i32, i32, C.POINTER(i32), C.POINTER(i32)]
        L.hago_probe_mfma_i8.restype = i32
        L.hago_probe_mfma_i8.argtypes = [vp, vp, i32, i32, vp]
        L.hago_probe_copy.restype = i32
        L.hago_probe_copy.argtypes = [vp, vp, i64, vp]
        L.hago_set_test_hook.restype = None
        L.hago_set_test_hook.argtypes = [i32, i32]
        _lib = L
    return _lib


def bit_range(bits, is_signed):
    """hago_bit_range: the inclusive code range of `bits` effective bits."""
    lo, hi = C.c_int32(), C.c_int32()
    _check(lib().hago_bit_range(int(bits), int(bool(is_signed)), C.byref(lo), C.byref(hi)))
    return lo.value, hi.value


def probe_mfma_i8(operands, sink, workgroups, iters):
    """hago_probe_mfma_i8: operands 8192 bytes, sink 4 bytes (device tensors)."""
    assert operands.numel() * operands.element_size() >= 8192 and sink.numel() * sink.element_size() >= 4
    _check(lib().hago_probe_mfma_i8(_ptr(operands), _ptr(sink), int(workgroups), int(iters), _stream()))


def probe_copy(src, dst):
    """hago_probe_copy between two device tensors of the same byte size."""
    n = src.numel() * src.element_size()
    assert n == dst.numel() * dst.element_size()
    _check(lib().hago_probe_copy(_ptr(src), _ptr(dst), n, _stream()))


def set_test_hook(key, value):
    """hago_set_test_hook: force a GEMM kernel family / tile for the following calls (tests)."""
    lib().hago_set_test_hook(int(key), int(value))


def _check(code):
    if code != 0:
        raise HagoError(code, lib().hago_status_string(code).decode())


class QType:
    """Container dtype, effective bits, signedness of the effective range, zero point."""

    def __init__(self, dtype, bits=None, is_signed=None, zero_point=0):
        self.dtype = dtype
        self.bits = {U8: 8, I8: 8, I16: 16, I32: 32, I24: 24}.get(dtype, 0) if bits is None else bits
        self.is_signed = (dtype != U8) if is_signed is None else bool(is_signed)
        self.zero_point = int(zero_point)

    def c(self):
        return _QType(self.dtype, self.bits, int(self.is_signed), self.zero_point)


class Requant:
    """Requantize parameters; multiplier/shift are int32 device tensors (multiplier None: the
    shift-only form for power-of-two scales)."""

    def __init__(self, multiplier, shift, out: QType, clip_lo=None, clip_hi=None, per_channel=None,
                 rounding=0):
        self.multiplier = multiplier
        self.shift = shift
        self.out = out
        lo, hi = bit_range(out.bits, out.is_signed)
        self.clip_lo = lo if clip_lo is None else int(clip_lo)
        self.clip_hi = hi if clip_hi is None else int(clip_hi)
        self.per_channel = int(shift.numel() > 1) if per_channel is None else int(per_channel)
        self.rounding = int(rounding)   # ROUND_UPWARD or ROUND_HALF_AWAY

    def c(self):
        return _Requant(None if self.multiplier is None else self.multiplier.data_ptr(), self.shift.data_ptr(), self.per_channel,
                        self.out.c(), self.clip_lo, self.clip_hi, self.rounding)


def _native_module():
    """The marshalling module (csrc/native.cpp), bound to the loaded library."""
    global _native
    if _native is None:
        L = lib()
        import torch  # noqa: F401  (the module links to torch's libraries)
        if not os.path.exists(_NATIVE_PATH):
            raise FileNotFoundError(
                f"{_NATIVE_PATH} is missing: build it with `python -m paper_2103_14949_amd.build` "
                "(there is no fallback path)")
        from . import _native as m
        m.bind({name: C.cast(getattr(L, name), C.c_void_p).value for name in m.entries()}, _check)
        _native = m
    return _native


def __getattr__(name):
    # the type of the calls that prepare=True returns
    if name == "Prepared":
        return _native_module().Prepared
    raise AttributeError(name)


def _stream():
    import torch
    return torch.cuda.current_stream().cuda_stream


def _ptr(t):
    return None if t is None else t.data_ptr()


# Every operator below takes its output tensor as `out` (allocated when None), launches on torch's current
# stream and returns the output; with prepare=True it returns instead a Prepared object, a call with its
# arguments already marshalled (`.out` is its output) that re-issues the same launch on the same buffers and stream.

def simquant(x, scale, zero_point, q: QType, clip_lo=None, clip_hi=None, per_channel=None, out=None,
             prepare=False):
    """hago_simquant over x[outer, channels, inner] (fp32, contiguous)."""
    return (_native or _native_module()).simquant(x, scale, zero_point, q, clip_lo, clip_hi, per_channel, out, prepare)


def simquant_wrap(x, scale, zero_point, q: QType, clip_lo=None, clip_hi=None, per_channel=None, out=None,
                  prepare=False):
    """hago_simquant_wrap over x[outer, channels, inner]: simulated quantize with the overflow of q's container."""
    return (_native or _native_module()).simquant_wrap(x, scale, zero_point, q, clip_lo, clip_hi, per_channel, out, prepare)


def simquant_batched(x, scales, zero_points, q: QType, clip_lo, clip_hi, per_channel=True, out=None,
                     prepare=False):
    """hago_simquant_batched: candidates b over x[outer, channels, inner]; scales / zero_points are
    device tensors [nbatch, channels] (or [nbatch, 1]); clip_lo / clip_hi are host sequences."""
    return (_native or _native_module()).simquant_batched(x, scales, zero_points, q, clip_lo, clip_hi, per_channel, out, prepare)


def quantize(x, scale, zero_point, q: QType, clip_lo=None, clip_hi=None, per_channel=None, out=None,
             prepare=False):
    """hago_quantize over x[outer, channels, inner] (fp32): integer codes in q's container."""
    return (_native or _native_module()).quantize(x, scale, zero_point, q, clip_lo, clip_hi, per_channel, out, prepare)


def simquant_codes(x, scale, zero_point, q: QType, clip_lo=None, clip_hi=None, per_channel=None, out=None,
                   out_codes=None, prepare=False):
    """hago_simquant_codes over x[outer, channels, inner] (fp32): (simulated-quantized fp32, integer codes)."""
    return (_native or _native_module()).simquant_codes(x, scale, zero_point, q, clip_lo, clip_hi, per_channel, out, out_codes,
                                                        prepare)


def dequantize(codes, q: QType, scale, zero_point, per_channel=None, out=None, prepare=False):
    """hago_dequantize over codes[outer, channels, inner] in q's container: fp32."""
    return (_native or _native_module()).dequantize(codes, q, scale, zero_point, per_channel, out, prepare)


def absmax(x, per_channel=True, out=None, prepare=False):
    """hago_absmax over x[outer, channels, inner] (fp32, contiguous): thresholds [channels] or [1]."""
    return (_native or _native_module()).absmax(x, per_channel, out, prepare)


def requantize(acc, rq: Requant, out=None, prepare=False):
    """hago_requantize over acc[outer, channels, inner] (int32 / int16)."""
    return (_native or _native_module()).requantize(acc, rq, out, prepare)


def qdense(a, a_t: QType, w, w_t: QType, bias=None, acc_dtype=I32, rq: Requant | None = None,
           flags=0, out=None, prepare=False):
    """hago_qdense: a [M,K] (uint8/int8), w [N,K] int8 -> [M,N].

    prepare=True returns a Prepared call instead of launching."""
    return (_native or _native_module()).qdense(a, a_t, w, w_t, bias, acc_dtype, rq, flags, out, prepare)


def _conv_dims(a, w, layout):
    if layout == NCHW:
        B, Cc, H, W = a.shape
        O, _, KH, KW = w.shape
    else:
        B, H, W, Cc = a.shape
        O, KH, KW, _ = w.shape
    return B, Cc, H, W, O, KH, KW


def qconv2d_workspace_bytes(a_shape, w_shape, layout=NCHW, stride=(1, 1), pad=(0, 0), groups=1):
    """hago_qconv2d_workspace_bytes for tensors of these shapes."""
    class _S:
        def __init__(self, shape):
            self.shape = tuple(shape)
    B, Cc, H, W, O, KH, KW = _conv_dims(_S(a_shape), _S(w_shape), layout)
    return int(lib().hago_qconv2d_workspace_bytes(layout, B, Cc, H, W, O, KH, KW, stride[0], stride[1],
                                                  pad[0], pad[1], groups))


def qconv2d(a, a_t: QType, w, w_t: QType, bias=None, layout=NCHW, stride=(1, 1), pad=(0, 0),
            groups=1, acc_dtype=I32, rq: Requant | None = None, flags=0, out=None, prepare=False,
            workspace=None, static_scratch=False):
    """hago_qconv2d: NCHW a [B,C,H,W], w [O,C/g,KH,KW]; NHWC a [B,H,W,C], w [O,KH,KW,C/g].

    With `workspace` (a uint8 device tensor of at least qconv2d_workspace_bytes(...) bytes, or an
    empty one when that is 0) the call goes to hago_qconv2d_ws; with static_scratch=True to
    hago_qconv2d_static."""
    return (_native or _native_module()).qconv2d(a, a_t, w, w_t, bias, layout, stride, pad, groups, acc_dtype, rq, flags, out,
                                                 prepare, workspace, static_scratch)
