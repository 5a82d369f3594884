"""Thin binding over libbmx.so: argument marshalling only.

Every function takes torch tensors that already live on the GPU (PyTorch is used for
device memory and streams, nothing else), passes raw device pointers and sizes through
the C ABI declared in include/bmx.h and raises BmxError on a non-zero status.  The layer
calls go through the native module _bmx_host (csrc/host_binding.cpp: the checks, the output
and workspace tensors, the call), the queries and hooks through ctypes.  There is
no CPU fallback: if the HIP library cannot be loaded the import of this module's
functions fails loudly on first use.
"""
import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libbmx.so")
HOST_PATH = os.path.join(_HERE, "_bmx_host.so")
_lib = None
_native = None

OP_BINARY_FC, OP_BINARY_CONV2D, OP_QUANT_GEMM, OP_BINARY_CONV2D_BITS, OP_XNOR_GEMM_W32 = 1, 2, 3, 4, 5
EXPORTS = ["bmx_binarize_pack", "bmx_xnor_gemm", "bmx_binary_fc", "bmx_pack_conv_weights",
           "bmx_binary_conv2d", "bmx_quant_gemm", "bmx_alpha_mean_abs", "bmx_pack_nchw",
           "bmx_binary_conv2d_packed", "bmx_workspace_bytes", "bmx_status_string", "bmx_version",
           "bmx_conv_weight_row_words", "bmx_binary_fc_packed", "bmx_tune_set",
           "bmx_binary_conv2d_bits", "bmx_xnor_gemm_count", "bmx_unpack_pm1", "bmx_widen_words32",
           "bmx_xnor_gemm_w32", "bmx_binary_fc_static", "bmx_last_kernel",
           "bmx_probe_valu"]

_i64, _int, _p, _sz = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t


class BmxError(RuntimeError):
    def __init__(self, status, what):
        self.status = status
        super().__init__("%s failed: %s" % (what, status_string(status)))


def lib():
    """Load libbmx.so (building it first only if no built library is present)."""
    global _lib
    if _lib is None:
        if not (os.path.exists(LIB_PATH) and os.path.exists(HOST_PATH)):
            from . import build as _build
            _build.build()
        # (global: the native module finds the library's entry points here)
        L = ctypes.CDLL(LIB_PATH, mode=ctypes.RTLD_GLOBAL)
        L.bmx_binarize_pack.argtypes = [_p, _i64, _i64, _i64, _int, _p, _i64, _p]
        L.bmx_xnor_gemm.argtypes = [_p, _i64, _p, _i64, _p, _i64, _int, _int, _int, _p]
        L.bmx_xnor_gemm_count.argtypes = L.bmx_xnor_gemm.argtypes
        L.bmx_unpack_pm1.argtypes = [_p, _i64, _i64, _i64, _p, _i64, _p]
        L.bmx_unpack_pm1.restype = _int
        L.bmx_xnor_gemm_count.restype = _int
        L.bmx_binary_fc.argtypes = [_p, _i64, _p, _i64, _p, _int, _int, _int, _p, _p, _i64, _p, _sz, _p]
        L.bmx_pack_conv_weights.argtypes = [_p, _int, _int, _int, _int, _p, _p]
        L.bmx_binary_conv2d.argtypes = [_p, _int, _int, _int, _int, _p, _int, _int, _int, _int, _int,
                                        _p, _p, _p, _p, _sz, _p]
        L.bmx_quant_gemm.argtypes = [_p, _i64, _int, _p, _i64, _int, _int, _int, _int, _p, _p, _i64,
                                     _p, _sz, _p]
        L.bmx_alpha_mean_abs.argtypes = [_p, _i64, _i64, _i64, _p, _p]
        L.bmx_workspace_bytes.argtypes = [_int, ctypes.POINTER(_i64), _int]
        L.bmx_workspace_bytes.restype = _sz
        L.bmx_status_string.argtypes = [_int]
        L.bmx_status_string.restype = ctypes.c_char_p
        L.bmx_version.restype = _int
        L.bmx_binary_fc_packed.argtypes = [_p, _i64, _p, _i64, _p, _int, _int, _int, _p, _p, _p, _p, _i64, _p]
        L.bmx_binary_fc_packed.restype = _int
        L.bmx_conv_weight_row_words.argtypes = [_int, _int, _int]
        L.bmx_conv_weight_row_words.restype = _i64
        L.bmx_pack_nchw.argtypes = [_p, _int, _int, _int, _int, _int, _p, _p]
        L.bmx_binary_conv2d_packed.argtypes = [_p, _int, _int, _int, _int, _p, _int, _int, _int, _int,
                                               _int, _p, _p, _p, _p]
        L.bmx_binary_conv2d_bits.argtypes = [_p, _int, _int, _int, _int, _p, _int, _int, _int, _int, _int,
                                             _p, _p, _p, _int, _p, _sz, _p]
        L.bmx_binary_conv2d_bits.restype = _int
        L.bmx_widen_words32.argtypes = [_p, _i64, _i64, _i64, _p, _i64, _p]
        L.bmx_widen_words32.restype = _int
        L.bmx_xnor_gemm_w32.argtypes = [_p, _i64, _p, _i64, _p, _i64, _int, _int, _int, _p, _sz, _p]
        L.bmx_xnor_gemm_w32.restype = _int
        L.bmx_binary_fc_static.argtypes = [_p, _i64, _p, _i64, _p, _int, _int, _int, _p, _p, _i64, _p]
        L.bmx_binary_fc_static.restype = _int
        L.bmx_last_kernel.restype = ctypes.c_char_p
        L.bmx_probe_valu.argtypes = [_int, _int, _p, ctypes.POINTER(_int), _p]
        L.bmx_probe_valu.restype = _int
        L.bmx_tune_set.argtypes = [_int, _int]
        L.bmx_tune_set.restype = _int
        for name in EXPORTS[:9]:
            getattr(L, name).restype = _int
        _lib = L
    return _lib


def _host():
    """The native module of the layer calls, on top of the loaded library."""
    global _native
    if _native is None:
        lib()
        from . import _bmx_host
        _bmx_host.set_error(BmxError)
        _native = _bmx_host
    return _native


def status_string(status):
    return lib().bmx_status_string(int(status)).decode()


def last_kernel():
    """Name and launch shape of the last compute kernel this thread launched through the library."""
    return lib().bmx_last_kernel().decode()


def probe_valu(workgroups, iters, out3, stream=None):
    """Launch the register-only xor+popcount chain; returns the wall-clock rate in kHz.  out3 is
    an int64 device tensor of 3 elements (cycles, wall ticks, sink)."""
    _chk(out3, _U64, "probe_valu out3", dense=True)
    khz = _int(0)
    _check(lib().bmx_probe_valu(int(workgroups), int(iters), _ptr(out3), ctypes.byref(khz), _stream(stream)),
           "bmx_probe_valu")
    return int(khz.value)


def version():
    return int(lib().bmx_version())


def _ptr(t):
    return _p(0) if t is None else _p(t.data_ptr())


_F32, _I32, _U64 = (torch.float32,), (torch.int32,), (torch.int64,)


def _chk(t, dtypes, what, dense=False):
    """Host-side guard in front of the C ABI, which sees only a raw address: the tensor must
    live on the GPU, have the element type the call reads or writes, and unit stride along its
    last dimension (rows may be further apart: the leading dimension is passed on).  With
    `dense` the whole tensor must be contiguous (layouts the C call takes no strides for)."""
    if t is None:
        return None
    if not hasattr(t, "data_ptr") or not hasattr(t, "is_cuda"):
        raise ValueError("%s: expected a torch tensor, got %s" % (what, type(t).__name__))
    if not t.is_cuda:
        raise ValueError("%s: tensor must live on the GPU (device is %s)" % (what, t.device))
    if t.dtype not in dtypes:
        raise ValueError("%s: dtype %s, expected %s" % (what, t.dtype, " or ".join(str(d) for d in dtypes)))
    if dense:
        if not t.is_contiguous():
            raise ValueError("%s: tensor must be contiguous" % what)
    elif t.dim() >= 1 and t.numel() > 1 and t.shape[-1] > 1 and t.stride(-1) != 1:
        raise ValueError("%s: last dimension must have stride 1 (got %d)" % (what, t.stride(-1)))
    elif t.dim() > 2 and not t.is_contiguous():
        raise ValueError("%s: tensor must be contiguous" % what)
    return t


def _ld(t):
    """Row stride of a 2-D tensor in elements (its row length when it has a single row)."""
    return t.stride(0) if t.shape[0] > 1 else max(t.shape[1], 1)


def _stream(stream):
    if stream is None:
        stream = torch.cuda.current_stream()
    return _p(stream.cuda_stream)


def _check(status, what):
    if status != 0:
        raise BmxError(status, what)


def workspace_bytes(op, dims):
    arr = (_i64 * len(dims))(*[int(d) for d in dims])
    return int(lib().bmx_workspace_bytes(int(op), arr, len(dims)))


def binarize_pack(x, pack_dim=1, out=None, stream=None):
    """x: fp32 [rows, cols] device tensor (row-major, stride(1) == 1).  Returns packed int64
    storage [R, ceil(K/64)] holding the uint64 words."""
    return (_native or _host()).binarize_pack(x, pack_dim, out, stream)


def unpack_pm1(bits, K, out=None, stream=None):
    """bits: packed int64 storage [rows, words] -> fp32 [rows, K] of +1 / -1."""
    return (_native or _host()).unpack_pm1(bits, K, out, stream)


def xnor_gemm(A, B, K, out=None, stream=None, count=False):
    """count: the xnor count (dot + K) / 2 of Eq. 2 instead of the dot product."""
    return (_native or _host()).xnor_gemm(A, B, K, out, stream, count)


def widen_words32(rows32, K, out=None, stream=None):
    """rows32: int32 storage [rows, dwords] holding rows of 32-bit words (the 32-bit BINARY_WORD
    flavour) -> int64 storage [rows, ceil(K/64)] holding the same rows as 64-bit words."""
    return (_native or _host()).widen_words32(rows32, K, out, stream)


def xnor_gemm_w32(A32, B32, K, out=None, workspace=None, stream=None):
    """bmx_xnor_gemm on operands stored as rows of 32-bit words (int32 storage)."""
    return (_native or _host()).xnor_gemm_w32(A32, B32, K, out, workspace, stream)


def binary_fc(x, Wp, alpha=None, integer_out=False, out=None, workspace=None, stream=None):
    return (_native or _host()).binary_fc(x, Wp, alpha, integer_out, out, workspace, stream)


def binary_fc_static(x, Wp, alpha=None, integer_out=False, out=None, stream=None):
    """bmx_binary_fc on the library's own scratch array: the call itself allocates nothing, so
    `out` must be given."""
    return (_native or _host()).binary_fc_static(x, Wp, alpha, integer_out, out, stream)


def binary_fc_packed(xp, in_features, Wp, alpha=None, mode="f32", out=None, thr=None, stream=None):
    """xp: packed activations [batch, words]; like every packed matrix here and every given out it may be a
    contiguous tensor of more dimensions, e.g. a packed image [N, H, W, words] as N rows.  mode: "f32", "i32" or "bits" (packed sign bits,
    against the per-feature threshold thr if given)."""
    return (_native or _host()).binary_fc_packed(xp, in_features, Wp, alpha, mode, out, thr, stream)


def pack_conv_weights(w, stream=None):
    return (_native or _host()).pack_conv_weights(w, stream)


def conv_out_hw(H, W, KH, KW, stride, pad):
    return (H + 2 * pad - KH) // stride + 1, (W + 2 * pad - KW) // stride + 1


def binary_conv2d(x, Wp, O, KH, KW, stride=1, pad=0, alpha=None, integer_out=False, out=None,
                  workspace=None, stream=None):
    return (_native or _host()).binary_conv2d(x, Wp, O, KH, KW, stride, pad, alpha, integer_out, out, workspace, stream)


def pack_nchw(x, pad=0, out=None, stream=None):
    return (_native or _host()).pack_nchw(x, pad, out, stream)


def binary_conv2d_packed(xp, C, Wp, O, KH, KW, stride=1, pad=0, alpha=None, integer_out=False,
                         out=None, stream=None):
    return (_native or _host()).binary_conv2d_packed(xp, C, Wp, O, KH, KW, stride, pad, alpha, integer_out, out, stream)


def binary_conv2d_bits(xp, C, Wp, O, KH, KW, stride=1, pad=0, alpha=None, thr=None, out_pad=1,
                       out=None, workspace=None, stream=None):
    """Convolution on a packed image whose result is the next convolution's packed image
    [N, Ho + 2*out_pad, Wo + 2*out_pad, ceil(O/64)] (int64 storage holding the uint64 words)."""
    return (_native or _host()).binary_conv2d_bits(xp, C, Wp, O, KH, KW, stride, pad, alpha, thr, out_pad, out,
                                                   workspace, stream)


def quant_gemm(a, w, bits_a, bits_w=1, want_int=True, want_float=True, out_int=None, out_float=None,
               workspace=None, stream=None):
    return (_native or _host()).quant_gemm(a, w, bits_a, bits_w, want_int, want_float, out_int, out_float, workspace, stream)


def alpha_mean_abs(w, stream=None):
    return (_native or _host()).alpha_mean_abs(w, stream)
