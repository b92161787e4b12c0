"""Binding of ``libjetfire.so``: same names as the C ABI, argument marshalling only.

The operators go through the extension module ``_native`` (csrc/jf_python.cpp), which checks the tensors, allocates the
outputs and launches in C++: for small layers the host's share of a call is what bounds it.  ``load_library()`` is the
C ABI itself through ctypes.  torch is used for device memory and the current stream; nothing here computes.
"""
import ctypes
import importlib
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libjetfire.so")
_EXT_PATH = os.path.join(_HERE, "_native.so")
_lib = None
_ext = None

# name -> argument ctypes, in the order of include/jetfire.h
_P, _I64, _I32, _F32, _SZ = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_float, ctypes.c_size_t
_SIGNATURES = {
    "jf_last_hip_error": (_I32, []),
    "jf_error_string": (ctypes.c_char_p, [_I32]),
    "jf_workspace_bytes": (_SZ, [_I32, _I64, _I64, _I64, _I32]),
    "jf_quantize_block": (_I32, [_P, _I32, _I64, _I64, _I64, _I32, _P, _I64, _P, _P, _I64, _P, _P]),
    "jf_dequantize_block": (_I32, [_P, _P, _I64, _I64, _I32, _P, _I32, _I64, _P]),
    "jf_linear_fwd": (_I32, [_P, _P, _P, _P, _I64, _I64, _I64, _I32, _P, _P, _P, _P, _SZ, _P]),
    "jf_linear_dgrad": (_I32, [_P, _P, _P, _P, _I64, _I64, _I64, _I32, _P, _P, _P, _P, _SZ, _P]),
    "jf_linear_wgrad": (_I32, [_P, _P, _P, _P, _I64, _I64, _I64, _I32, _P, _P, _P, _P, _SZ, _P]),
    "jf_linear_bwd": (_I32, [_P, _P, _P, _P, _P, _P, _I64, _I64, _I64, _I32, _P, _P, _P, _P, _P, _P, _P, _SZ, _P]),
    "jf_gelu_q": (_I32, [_P, _P, _I64, _I64, _I32, _P, _P, _P]),
    "jf_gelu_q_bwd": (_I32, [_P, _P, _P, _P, _I64, _I64, _I32, _P, _P, _P]),
    "jf_layernorm_q": (_I32, [_P, _P, _P, _P, _F32, _I64, _I64, _I32, _P, _P, _P, _P, _P]),
    "jf_layernorm_q_partials": (_I32, [_P, _P, _P, _P, _P, _P, _F32, _I64, _I64, _I32, _P, _P, _P, _P, _P]),
    "jf_dropout_q": (_I32, [_P, _P, _P, _F32, _I64, _I64, _I32, _P, _P, _P]),
    "jf_add_q": (_I32, [_P, _P, _P, _P, _I64, _I64, _I32, _P, _P, _P, _P, _P]),
    "jf_layernorm_q_bwd": (_I32, [_P, _P, _P, _P, _P, _P, _P, _I64, _I64, _I32, _P, _P, _P, _P, _P, _SZ, _P]),
    "jf_layernorm_q_bwd_static": (_I32, [_P, _P, _P, _P, _P, _P, _P, _I64, _I64, _I32, _P, _P, _P, _P, _P]),
    "jf_debug_linear_partials": (_I32, [_I32, _P, _P, _I64, _I64, _I64, _I32, _I64, _P, _P]),
    "jf_debug_set_gemm_shape": (_I32, [_I32]),
}
EXPORTED_SYMBOLS = tuple(_SIGNATURES)

JF_OP_QUANTIZE, JF_OP_LINEAR_FWD, JF_OP_LINEAR_DGRAD, JF_OP_LINEAR_WGRAD = 0, 1, 2, 3
JF_OP_GELU, JF_OP_GELU_BWD, JF_OP_LAYERNORM, JF_OP_LAYERNORM_BWD = 4, 5, 6, 7


class JetfireError(RuntimeError):
    def __init__(self, code, message):
        super().__init__(message)
        self.code = code


def library_path() -> str:
    return _LIB_PATH


def load_library():
    """Load the built shared object; raises if it has not been built (there is no fallback path)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise JetfireError(-1, f"{_LIB_PATH} is missing: run `python -m paper_2403_12422_amd.build` "
                                   "(or __graft_entry__.build()) first; there is no CPU fallback")
        lib = ctypes.CDLL(_LIB_PATH)
        for name, (res, args) in _SIGNATURES.items():
            fn = getattr(lib, name)
            fn.restype = res
            fn.argtypes = args
        _lib = lib
    return _lib


def _native():
    """The extension module; it links the library, so that is what has to be there first."""
    global _ext
    if _ext is None:
        load_library()
        if not os.path.exists(_EXT_PATH):
            raise JetfireError(-1, f"{_EXT_PATH} is missing: run `python -m paper_2403_12422_amd.build` with the headers of this "
                                   "Python and torch installed; without it only load_library() works, the C ABI itself")
        ext = importlib.import_module(__package__ + "._native")
        ext.init(JetfireError)
        _ext = ext
    return _ext


def _check(code):
    if code != 0:
        lib = load_library()
        msg = lib.jf_error_string(code).decode()
        if code == 6:
            msg += f" (hip error {lib.jf_last_hip_error()})"
        raise JetfireError(code, msg)


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _dev(t, dtype, ndim):
    if not t.is_cuda:
        raise JetfireError(-2, "tensors must live on the GPU; this library has no CPU path")
    if t.dtype != dtype or t.dim() != ndim or not t.is_contiguous():
        raise JetfireError(-2, f"expected contiguous {ndim}-d {dtype} tensor, got {t.dtype} {tuple(t.shape)}")
    return t


def jf_workspace_bytes(op, N, C, D, block):
    return int(load_library().jf_workspace_bytes(op, N, C, D, block))


def jf_quantize_block(x, block=32, transposed_copy=False, out=None):
    """x: (rows, cols) float32 or float16 CUDA tensor -> (q, s) or (q, s, qT, sT).

    `out` (here and in every function below) is an optional tuple of preallocated output tensors, in the
    order they are returned; without it the outputs are allocated with torch."""
    return (_ext or _native()).quantize(x, block, transposed_copy, out)


def jf_dequantize_block(q, s, block=32, dtype=torch.float32, out=None):
    """(codes, scales) -> float32 or float16 tensor of code * scale."""
    if dtype not in (torch.float32, torch.float16):
        raise JetfireError(7, "output must be float32 or float16")
    return (_ext or _native()).dequantize(q, s, block, dtype == torch.float16, out)


def jf_linear_fwd(X, SX, W, SW, block=32, want_f32=False, out=None):
    """Y = X W^T.  X (N,C) int8, W (D,C) int8 -> (Y int8 (N,D), SY, Y_f32 or None)."""
    return (_ext or _native()).linear_fwd(X, SX, W, SW, block, want_f32, out)


def jf_linear_dgrad(dY, SdY, W, SW, block=32, want_f32=False, out=None):
    """dX = dY W.  dY (N,D) int8, W (D,C) int8 -> (dX int8 (N,C), SdX, dX_f32 or None)."""
    return (_ext or _native()).linear_dgrad(dY, SdY, W, SW, block, want_f32, out)


def jf_linear_wgrad(dY, SdY, X, SX, block=32, want_q=True, want_f32=False, out=None):
    """dW = dY^T X.  dY (N,D) int8, X (N,C) int8 -> (dW int8 (D,C) or None, SdW or None, dW_f32 or None)."""
    return (_ext or _native()).linear_wgrad(dY, SdY, X, SX, block, want_q, want_f32, out)


def jf_linear_bwd(dY, SdY, W, SW, X, SX, block=32, want_f32=False, out=None):
    """Both backward products in one call: returns ((dX, SdX, dX_f32 or None), (dW, SdW, dW_f32 or None)); `out` is the
    same pair of triples, preallocated."""
    return (_ext or _native()).linear_bwd(dY, SdY, W, SW, X, SX, block, want_f32, out)


def jf_gelu_q(X, SX, block=32, out=None):
    return (_ext or _native()).gelu(X, SX, block, out)


def jf_gelu_q_bwd(dY, SdY, X, SX, block=32, out=None):
    return (_ext or _native()).gelu_bwd(dY, SdY, X, SX, block, out)


def jf_layernorm_q(X, SX, gamma, beta, eps=1e-5, block=32, out=None):
    return (_ext or _native()).layernorm(X, SX, None, None, gamma, beta, eps, block, out)


def jf_layernorm_q_partials(X, SX, row_mean, row_sumsq, gamma, beta, eps=1e-5, block=32, out=None):
    """LayerNorm whose row statistics come from the row partials written by jf_add_q."""
    if row_mean is None or row_sumsq is None:
        raise JetfireError(1, "row_mean and row_sumsq are required")
    return (_ext or _native()).layernorm(X, SX, row_mean, row_sumsq, gamma, beta, eps, block, out)


def jf_dropout_q(X, SX, mask_bits, p, block=32, out=None):
    """Y = Q(X * m / (1 - p)); mask_bits (N, C/8) uint8, bit c % 8 of byte c // 8 of a row is column c's keep bit."""
    return (_ext or _native()).dropout(X, SX, mask_bits, p, block, out)


def jf_add_q(X1, S1, X2, S2, block=32, want_partials=False, out=None):
    """Y = Q(X1 + X2); with want_partials also the row partials (mean, sum of squares) of the sum, stored block column by
    block column: two (C/block, N) tensors."""
    return (_ext or _native()).add(X1, S1, X2, S2, block, want_partials, out)


def jf_layernorm_q_bwd(dY, SdY, X, SX, gamma, mean, rstd, block=32, workspace=None, out=None):
    return (_ext or _native()).layernorm_bwd(dY, SdY, X, SX, gamma, mean, rstd, block, workspace, out, False)


def jf_layernorm_q_bwd_static(dY, SdY, X, SX, gamma, mean, rstd, out, block=32):
    """jf_layernorm_q_bwd without a workspace: the library's static device scratch holds the partial sums, and
    nothing is allocated -- `out` = (dX, SdX, dgamma, dbeta), preallocated, is therefore required."""
    return (_ext or _native()).layernorm_bwd(dY, SdY, X, SX, gamma, mean, rstd, block, None, out, True)


def jf_debug_linear_partials(which, A, Bm, N, C, D, block, kb):
    """INT32 product of K-block kb (test hook); which: 0 fwd, 1 dgrad, 2 wgrad."""
    _dev(A, torch.int8, 2), _dev(Bm, torch.int8, 2)
    shape = {0: (N, D), 1: (N, C), 2: (D, C)}[which]
    out = torch.empty(shape, dtype=torch.int32, device=A.device)
    _check(load_library().jf_debug_linear_partials(which, _ptr(A), _ptr(Bm), N, C, D, block, kb, _ptr(out), _stream()))
    return out


def jf_debug_set_gemm_shape(shape):
    """Test hook: 0 automatic, 1 128x128, 4 64x64, 6 256x128, 8 128x64, 10 32x32, 21..25 pairs of shapes for both backward
    products in one launch, as far as the block size has them (include/jetfire.h); else the choice stays automatic."""
    _check(load_library().jf_debug_set_gemm_shape(shape))
