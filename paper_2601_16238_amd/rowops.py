"""Thin binding of the row-wise entry points of include/rowops.h (RMSNorm forward, LayerNorm
forward and backward, rotary forward): argument marshalling only (csrc/marshal.cpp), every step
runs in the HIP kernels of libmi355attn.so."""
import ctypes

from .binding import _call, lib, marshal

EXPORTS = ("rowops_rmsnorm_fwd", "rowops_layernorm_fwd", "rowops_layernorm_bwd_workspace_bytes",
           "rowops_layernorm_bwd", "rowops_rotary_fwd")
_bound = False


def _lib():
    global _bound
    L = lib()
    if not _bound:
        vp, i32, i64, f32 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_float
        L.rowops_rmsnorm_fwd.argtypes = [vp, vp, vp, i64, i32, i64, i64, f32, vp]
        L.rowops_layernorm_fwd.argtypes = [vp, vp, vp, vp, vp, vp, i64, i32, i64, i64, f32, vp]
        L.rowops_layernorm_bwd_workspace_bytes.argtypes = [i64, i32]
        L.rowops_layernorm_bwd_workspace_bytes.restype = ctypes.c_size_t
        L.rowops_layernorm_bwd.argtypes = [vp] * 8 + [vp, ctypes.c_size_t, i64, i32, i64, i64, i64, vp]
        L.rowops_rotary_fwd.argtypes = [vp, vp, vp, vp, i32, i32, i32, i32] + [i64] * 6 + [vp]
        for n in ("rowops_rmsnorm_fwd", "rowops_layernorm_fwd", "rowops_layernorm_bwd",
                  "rowops_rotary_fwd"):
            getattr(L, n).restype = ctypes.c_int
        _bound = True
    return L


def rmsnorm_fwd(x, w, eps, y=None, stream=None):
    return _call(marshal().rmsnorm_fwd, stream, x, w, eps, y)


def layernorm_fwd(x, w, b, eps, y=None, mean=None, rstd=None, stream=None):
    return _call(marshal().layernorm_fwd, stream, x, w, b, eps, y, mean, rstd)


def layernorm_bwd_workspace_bytes(rows, cols):
    return int(_lib().rowops_layernorm_bwd_workspace_bytes(rows, cols))


def layernorm_bwd(dy, x, w, mean, rstd, dx=None, dw=None, db=None, workspace=None, stream=None):
    return _call(marshal().layernorm_bwd, stream, dy, x, w, mean, rstd, dx, dw, db, workspace)


def rotary_fwd(x, cos, sin, y=None, stream=None):
    return _call(marshal().rotary_fwd, stream, x, cos, sin, y)
