"""The library's internal convolution calls, for what the layer calls leave out: BN sums, addends, masks, prepared filters."""
import ctypes as C

import torch

from paper_2107_00961_amd import binding as B

_CONV_FWD = "_ZN6resist8conv_fwdERKNS_8ConvGeomEiPKvRKNS_6FilterEPvS4_PfPNS_9StatPartsEP12ihipStream_tPKNS_7EvalActE"
_CONV_WGRAD = "_ZN6resist10conv_wgradERKNS_8ConvGeomEiPKvS4_PfS5_P12ihipStream_tb"
_WGRAD_SCRATCH = "_ZN6resist20wgrad_scratch_floatsERKNS_8ConvGeomEib"
_CONV_DGRAD = "_ZN6resist10conv_dgradERKNS_8ConvGeomEiPKvRKNS_6FilterEPvS4_S4_P12ihipStream_tPKNS_9BnBwdFuseE"


class Geom(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("N", "H", "W", "C", "K", "R", "S", "stride", "pad", "P", "Q")]


class Filter(C.Structure):
    _fields_ = [("w", C.c_void_p), ("prep", C.c_void_p), ("fragments", C.c_bool), ("scale", C.c_float)]


class StatParts(C.Structure):
    _fields_ = [("parts", C.c_int), ("rows", C.c_int)]


class BnBufs(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("gamma", "beta", "rmean", "rvar", "mean", "invstd", "scale", "shift", "dgamma", "dbeta")]


class BnBwdFuse(C.Structure):
    _fields_ = [("y", C.c_void_p), ("b", BnBufs), ("relu_of_self", C.c_bool), ("sums", C.c_void_p), ("parts", C.POINTER(StatParts))]


def geom(N, H, W, Cc, K, R, stride, pad):
    return Geom(N, H, W, Cc, K, R, R, stride, pad, (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1)


def _ptr(t):
    return C.c_void_p(t.data_ptr() if t is not None else None)


def conv_fwd(g, dtype, x, w, y, stats=None, prep=None):
    """-> (parts, rows): `stats` [3][parts][K] holds that many ranges of that many output pixels.  prep: w in matrix fragments."""
    sp = StatParts()
    f = Filter(w.data_ptr(), prep.data_ptr() if prep is not None else None, prep is not None, 1.0)
    B._check(B.lib()[_CONV_FWD](C.byref(g), dtype, _ptr(x), C.byref(f), _ptr(y), None, _ptr(stats), C.byref(sp), None, None))
    return sp.parts, sp.rows


def conv_dgrad(g, dtype, dy, wT, dx, addend=None, mask=None, bn=None):
    """wT [C][R][S][K].  bn: dict of y, mean, invstd, scale, shift, self, sums -> (parts, rows) of sums [2][parts][C]."""
    sp, f = StatParts(), None
    if bn is not None:
        bufs = BnBufs(mean=bn["mean"].data_ptr(), invstd=bn["invstd"].data_ptr(), scale=bn["scale"].data_ptr(), shift=bn["shift"].data_ptr())
        f = BnBwdFuse(bn["y"].data_ptr(), bufs, bn["self"], bn["sums"].data_ptr(), C.pointer(sp))
    B._check(B.lib()[_CONV_DGRAD](C.byref(g), dtype, _ptr(dy), C.byref(Filter(None, wT.data_ptr(), False, 1.0)), _ptr(dx), _ptr(addend), _ptr(mask), None,
                                  C.byref(f) if f is not None else None))
    return sp.parts, sp.rows


def conv_wgrad(g, dtype, dy, x, step):
    """dw [K][R][S][C], as a call on its own computes it or as a step does."""
    scratch = B.lib()[_WGRAD_SCRATCH]
    scratch.restype = C.c_int64
    part = torch.empty(max(1, scratch(C.byref(g), dtype, C.c_bool(step))), device="cuda")
    dw = torch.empty(g.K, g.R, g.S, g.C, device="cuda")
    B._check(B.lib()[_CONV_WGRAD](C.byref(g), dtype, _ptr(dy), _ptr(x), _ptr(dw), _ptr(part), None, C.c_bool(step)))
    return dw


def workspace(shape, bf16):
    """What the layer calls are told to bring for (N, H, W, C, K, R, stride, pad)."""
    return B._conv_ws(B._conv_shape(*shape, int(bf16)))


def _bytes(ws):
    return (_ptr(ws), ws.numel() * ws.element_size()) if ws is not None else (None, 0)


def forward_call(shape, x, w, ws):
    N, H, W, _, K, _, stride, pad = shape
    y = torch.empty((N, (H + 2 * pad - shape[5]) // stride + 1, (W + 2 * pad - shape[5]) // stride + 1, K), device="cuda", dtype=x.dtype)
    sh = B._conv_shape(*shape, int(x.dtype == torch.bfloat16))
    B._check(B.lib().resist_conv2d_forward(C.byref(sh), _ptr(x), _ptr(w), _ptr(y), *_bytes(ws), None))
    return y


def dgrad_call(shape, dy, w, ws):
    dx = torch.empty(shape[:4], device="cuda", dtype=dy.dtype)
    sh = B._conv_shape(*shape, int(dy.dtype == torch.bfloat16))
    B._check(B.lib().resist_conv2d_dgrad(C.byref(sh), _ptr(dy), _ptr(w), _ptr(dx), *_bytes(ws), None))
    return dx
