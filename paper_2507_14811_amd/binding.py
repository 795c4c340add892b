"""Thin ctypes binding of libsegquant.so: same names as the C ABI, argument marshalling only.

Every step of the path runs in the HIP kernels.  Device buffers are torch tensors (memory and
streams only); there is no CPU fallback: a missing library raises.
"""
from __future__ import annotations

import ctypes as C
import os
from typing import Optional, Sequence

import numpy as np

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libsegquant.so")

SQ_OK, SQ_ERR_INVALID_ARG, SQ_ERR_UNSUPPORTED, SQ_ERR_LAUNCH = 0, 1, 2, 3
SQ_F32, SQ_BF16 = 0, 1
SQ_MAX_SEGMENTS = 64
SQ_MAX_SEG_SCALE = 512
SQ_MAX_KSEG_LEN = 133143

EXPORTS = ("sq_quantize_weight", "sq_quantize_act", "sq_seglinear", "sq_seglinear_debug_acc",
           "sq_status_string", "sq_version", "sq_tuning_set", "sq_seglinear_grouped",
           "sq_quantize_weight_block", "sq_calibrate_act", "sq_calibrate_act_percentile",
           "sq_calibrate_workspace_bytes", "sq_quantize_act_fused",
           "sq_quantize_act_fused_workspace_bytes", "sq_quantize_weight_w4", "sq_seglinear_w4",
           "sq_seglinear_w4_debug_acc", "sq_quantize_act_dynamic", "sq_seglinear_dynamic",
           "sq_seglinear_fused", "sq_seglinear_grouped_fused", "sq_quantize_act_geglu",
           "sq_seglinear_fused_dynamic", "sq_unpack_w4", "sq_quantize_act_dynamic_bits", "sq_seglinear_grouped_w4",
           "sq_calibrate_act_percentile_static", "sq_calibrate_static_scratch_bytes",
           "sq_calibrate_channel_amax", "sq_weight_channel_amax", "sq_smooth_factors", "sq_quantize_weight_smoothed",
           "sq_quantize_act_smoothed", "sq_lowrank_add", "sq_lowrank_workspace_bytes",
           "sq_quantize_weight_fp8", "sq_quantize_act_fp8", "sq_seglinear_fp8", "sq_seglinear_grouped_fp8", "sq_quantize_act_fp8_fused")


class SqError(RuntimeError):
    def __init__(self, status: int, what: str):
        self.status = status
        super().__init__(f"{what}: {status_string(status)}")


class sq_group_item(C.Structure):
    _fields_ = [("wq", C.c_void_p), ("wscale", C.c_void_p), ("bias", C.c_void_p), ("y", C.c_void_p)]


class sq_layer(C.Structure):
    _fields_ = [
        ("M", C.c_int32), ("K", C.c_int32), ("N", C.c_int32),
        ("S", C.c_int32), ("kseg_off", C.POINTER(C.c_int32)),
        ("T", C.c_int32), ("nseg_off", C.POINTER(C.c_int32)),
        ("dual", C.POINTER(C.c_uint8)),
        ("s_pos", C.POINTER(C.c_float)), ("s_neg", C.POINTER(C.c_float)),
        ("seg_scale", C.POINTER(C.c_float)),
    ]


_lib = None


def load_library() -> C.CDLL:
    """Load libsegquant.so (built in-tree by paper_2507_14811_amd.build).  Raises if it is missing."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2507_14811_amd.build` "
                           "(there is no CPU fallback)")
    import torch  # noqa: F401  loads the HIP runtime the library binds to

    lib = C.CDLL(LIB_PATH)
    vp, i32 = C.c_void_p, C.c_int
    lp = C.POINTER(sq_layer)
    lib.sq_quantize_weight.argtypes = [lp, vp, i32, vp, vp, vp]
    lib.sq_quantize_act.argtypes = [lp, vp, i32, vp, vp]
    lib.sq_seglinear.argtypes = [lp, vp, vp, vp, vp, vp, i32, vp]
    lib.sq_seglinear_debug_acc.argtypes = [lp, vp, vp, vp, vp, vp]
    for f in (lib.sq_quantize_weight, lib.sq_quantize_act, lib.sq_seglinear, lib.sq_seglinear_debug_acc):
        f.restype = i32
    lib.sq_quantize_weight_block.argtypes = [lp, vp, i32, vp, vp, vp]
    lib.sq_quantize_weight_block.restype = i32
    lib.sq_calibrate_act.argtypes = [lp, vp, i32, vp, vp, i32, vp]
    lib.sq_calibrate_act.restype = i32
    lib.sq_quantize_act_fused.argtypes = [lp, vp, i32, C.POINTER(C.c_int32), vp, vp, C.c_size_t, vp]
    lib.sq_quantize_act_fused_workspace_bytes.argtypes = [lp]
    lib.sq_quantize_act_fused_workspace_bytes.restype = C.c_size_t
    lib.sq_quantize_act_fused.restype = i32
    lib.sq_quantize_weight_w4.argtypes = [lp, vp, i32, vp, vp, vp]
    lib.sq_seglinear_w4.argtypes = [lp, vp, vp, vp, vp, vp, i32, vp]
    lib.sq_seglinear_w4_debug_acc.argtypes = [lp, vp, vp, vp, vp, vp]
    for f in (lib.sq_quantize_weight_w4, lib.sq_seglinear_w4, lib.sq_seglinear_w4_debug_acc):
        f.restype = i32
    lib.sq_quantize_act_dynamic.argtypes = [lp, vp, i32, vp, vp, vp]
    lib.sq_quantize_act_dynamic.restype = i32
    lib.sq_seglinear_dynamic.argtypes = [lp, vp, vp, vp, i32, vp, vp, vp, i32, vp]
    lib.sq_seglinear_dynamic.restype = i32
    lib.sq_calibrate_act_percentile.argtypes = [lp, vp, i32, C.c_double, vp, vp, vp, C.c_size_t, i32, vp]
    lib.sq_calibrate_act_percentile.restype = i32
    lib.sq_calibrate_act_percentile_static.argtypes = [lp, vp, i32, C.c_double, vp, vp, i32, vp]
    lib.sq_calibrate_act_percentile_static.restype = i32
    lib.sq_calibrate_static_scratch_bytes.argtypes = []
    lib.sq_calibrate_static_scratch_bytes.restype = C.c_size_t
    lib.sq_calibrate_channel_amax.argtypes = [lp, vp, i32, vp, i32, vp]
    lib.sq_weight_channel_amax.argtypes = [lp, vp, i32, vp, vp]
    lib.sq_smooth_factors.argtypes = [lp, vp, vp, vp, vp, vp]
    lib.sq_quantize_weight_smoothed.argtypes = [lp, vp, i32, vp, vp, vp, vp]
    lib.sq_quantize_act_smoothed.argtypes = [lp, vp, i32, vp, vp, vp]
    for f in (lib.sq_calibrate_channel_amax, lib.sq_weight_channel_amax, lib.sq_smooth_factors,
              lib.sq_quantize_weight_smoothed, lib.sq_quantize_act_smoothed):
        f.restype = i32
    lib.sq_lowrank_add.argtypes = [lp, vp, i32, vp, vp, i32, vp, vp, i32, vp, C.c_size_t, vp]
    lib.sq_lowrank_add.restype = i32
    lib.sq_quantize_weight_fp8.argtypes = [lp, vp, i32, vp, vp, vp]
    lib.sq_quantize_weight_fp8.restype = i32
    lib.sq_quantize_act_fp8.argtypes = [lp, vp, i32, vp, vp]
    lib.sq_quantize_act_fp8.restype = i32
    lib.sq_quantize_act_fp8_fused.argtypes = [lp, vp, i32, C.POINTER(C.c_int32), vp, vp, C.c_size_t, vp]
    lib.sq_quantize_act_fp8_fused.restype = i32
    lib.sq_seglinear_fp8.argtypes = [lp, vp, vp, vp, vp, vp, i32, vp]
    lib.sq_seglinear_fp8.restype = i32
    lib.sq_lowrank_workspace_bytes.argtypes = [lp, i32]
    lib.sq_lowrank_workspace_bytes.restype = C.c_size_t
    lib.sq_calibrate_workspace_bytes.argtypes = []
    lib.sq_calibrate_workspace_bytes.restype = C.c_size_t
    lib.sq_seglinear_grouped.argtypes = [lp, vp, i32, C.POINTER(sq_group_item), i32, vp]
    lib.sq_seglinear_grouped.restype = i32
    lib.sq_seglinear_grouped_fp8.argtypes = [lp, vp, i32, C.POINTER(sq_group_item), i32, vp]
    lib.sq_seglinear_grouped_fp8.restype = i32
    lib.sq_quantize_act_geglu.argtypes = [lp, vp, i32, vp, vp]
    lib.sq_quantize_act_geglu.restype = i32
    lib.sq_seglinear_fused.argtypes = [lp, vp, i32, C.POINTER(C.c_int32), vp, vp, vp, vp, i32, vp]
    lib.sq_seglinear_fused.restype = i32
    lib.sq_unpack_w4.argtypes = [lp, vp, vp, vp]
    lib.sq_unpack_w4.restype = i32
    lib.sq_seglinear_fused_dynamic.argtypes = [lp, vp, i32, C.POINTER(C.c_int32), i32, vp, i32, vp, vp, vp, i32, vp]
    lib.sq_quantize_act_dynamic_bits.argtypes = [lp, vp, i32, i32, vp, vp, vp]
    lib.sq_quantize_act_dynamic_bits.restype = i32
    lib.sq_seglinear_fused_dynamic.restype = i32
    lib.sq_seglinear_grouped_w4.argtypes = [lp, vp, vp, i32, C.POINTER(sq_group_item), i32, vp]
    lib.sq_seglinear_grouped_w4.restype = i32
    lib.sq_seglinear_grouped_fused.argtypes = [lp, vp, i32, C.POINTER(C.c_int32), i32, C.POINTER(sq_group_item), i32, vp]
    lib.sq_seglinear_grouped_fused.restype = i32
    lib.sq_status_string.argtypes = [i32]
    lib.sq_status_string.restype = C.c_char_p
    lib.sq_version.restype = i32
    lib.sq_tuning_set.argtypes = [C.c_char_p, i32]
    lib.sq_tuning_set.restype = i32
    _lib = lib
    return lib


def status_string(status: int) -> str:
    return load_library().sq_status_string(int(status)).decode()


def sq_version() -> int:
    return int(load_library().sq_version())


def sq_tuning_set(key: str, value: int) -> None:
    st = load_library().sq_tuning_set(key.encode(), int(value))
    if st != SQ_OK:
        raise SqError(st, f"sq_tuning_set({key!r}, {value})")


class Layer:
    """Host-side descriptor (the C struct plus the numpy arrays that keep its pointers alive)."""

    def __init__(self, M: int, K: int, N: int, kseg_off: Sequence[int], nseg_off: Sequence[int],
                 dual: Sequence[int], s_pos=None, s_neg=None, seg_scale=None):
        self.kseg_off = np.ascontiguousarray(kseg_off, dtype=np.int32)
        self.nseg_off = np.ascontiguousarray(nseg_off, dtype=np.int32)
        self.dual = np.ascontiguousarray(dual, dtype=np.uint8)
        self.s_pos = None if s_pos is None else np.ascontiguousarray(s_pos, dtype=np.float32)
        self.s_neg = None if s_neg is None else np.ascontiguousarray(s_neg, dtype=np.float32)
        self.seg_scale = None if seg_scale is None else np.ascontiguousarray(seg_scale, dtype=np.float32)
        self.M, self.K, self.N = int(M), int(K), int(N)
        self.S, self.T = len(self.kseg_off) - 1, len(self.nseg_off) - 1

        def ptr(a, ty):
            return None if a is None else a.ctypes.data_as(C.POINTER(ty))

        self.c = sq_layer(self.M, self.K, self.N, self.S, ptr(self.kseg_off, C.c_int32), self.T,
                          ptr(self.nseg_off, C.c_int32), ptr(self.dual, C.c_uint8), ptr(self.s_pos, C.c_float),
                          ptr(self.s_neg, C.c_float), ptr(self.seg_scale, C.c_float))

    @classmethod
    def from_workload(cls, w) -> "Layer":
        return cls(w.M, w.K, w.N, w.kseg_off, w.nseg_off, w.dual, w.s_pos, w.s_neg, w.seg_scale)

    @property
    def any_dual(self) -> bool:
        return bool(self.dual.any())


# Host cost of a call: the small kernels take 3 - 8 us, so what a call costs in Python shows.  Addresses go to ctypes as
# plain integers (the argtypes say pointer), the current stream comes as its raw handle (torch.cuda.current_stream() builds
# an object for every call), and torch is looked up once.
_torch = None
_DTYPES: dict = {}


def _torch_module():
    global _torch
    if _torch is None:
        import torch

        _DTYPES.update({torch.float32: SQ_F32, torch.bfloat16: SQ_BF16})
        _torch = torch
    return _torch


def _dptr(t) -> Optional[int]:
    return None if t is None else t.data_ptr()


def _stream(stream):
    if stream is None:
        torch = _torch or _torch_module()
        if torch.cuda.is_initialized():
            return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
        stream = torch.cuda.current_stream()
    return getattr(stream, "cuda_stream", stream)


def _dt(t) -> int:
    if _torch is None:
        _torch_module()
    try:
        return _DTYPES[t.dtype]
    except KeyError:
        raise TypeError(f"unsupported dtype {t.dtype}") from None


def _check(st: int, what: str):
    if st != SQ_OK:
        raise SqError(st, what)


def sq_quantize_weight(layer: Layer, w, wq, wscale, stream=None) -> None:
    """w [N][K] fp32/bf16 -> wq int8 [N][K], wscale fp32 [S][N]  (device tensors, written in place)."""
    _check(load_library().sq_quantize_weight(C.byref(layer.c), _dptr(w), _dt(w), _dptr(wq), _dptr(wscale),
                                             _stream(stream)), "sq_quantize_weight")


def sq_quantize_weight_block(layer: Layer, w, wq, wscale, stream=None) -> None:
    """One step per (K-segment, N-segment) block: w [N][K] -> wq int8 [N][K], wscale fp32 [S][N] (constant per block)."""
    _check(load_library().sq_quantize_weight_block(C.byref(layer.c), _dptr(w), _dt(w), _dptr(wq), _dptr(wscale),
                                                   _stream(stream)), "sq_quantize_weight_block")


def sq_calibrate_act(layer: Layer, x, amax, steps, accumulate: bool = False, stream=None) -> None:
    """Min/max calibration over one batch: amax fp32 [2][S] running maxima (in/out), steps fp32 [2][S] (s_pos, s_neg)."""
    _check(load_library().sq_calibrate_act(C.byref(layer.c), _dptr(x), _dt(x), _dptr(amax), _dptr(steps),
                                           1 if accumulate else 0, _stream(stream)), "sq_calibrate_act")


def sq_calibrate_workspace_bytes() -> int:
    """Device bytes sq_calibrate_act_percentile needs as workspace."""
    return int(load_library().sq_calibrate_workspace_bytes())


def sq_calibrate_act_percentile(layer: Layer, x, p: float, amax, steps, workspace, accumulate: bool = False,
                                stream=None) -> None:
    """Percentile-clipping calibration over one batch (nearest-rank p-quantile per K-segment and polarity); amax,
    steps as sq_calibrate_act; workspace: a device byte tensor of at least sq_calibrate_workspace_bytes()."""
    _check(load_library().sq_calibrate_act_percentile(C.byref(layer.c), _dptr(x), _dt(x), float(p), _dptr(amax),
                                                      _dptr(steps), _dptr(workspace),
                                                      workspace.numel() * workspace.element_size(),
                                                      1 if accumulate else 0, _stream(stream)),
           "sq_calibrate_act_percentile")


def sq_calibrate_act_percentile_static(layer: Layer, x, p: float, amax, steps, accumulate: bool = False, stream=None) -> None:
    """sq_calibrate_act_percentile without a workspace: the select state lives in a static device array of the library
    (no allocation anywhere in the call; calls on one GPU must not overlap)."""
    _check(load_library().sq_calibrate_act_percentile_static(C.byref(layer.c), _dptr(x), _dt(x), float(p), _dptr(amax),
                                                             _dptr(steps), 1 if accumulate else 0, _stream(stream)),
           "sq_calibrate_act_percentile_static")


def sq_calibrate_channel_amax(layer: Layer, x, amax_k, accumulate: bool = False, stream=None) -> None:
    """Per-input-channel maxima of |x| over one batch into amax_k (device fp32 [K]), running over batches if asked."""
    _check(load_library().sq_calibrate_channel_amax(C.byref(layer.c), _dptr(x), _dt(x), _dptr(amax_k),
                                                    1 if accumulate else 0, _stream(stream)), "sq_calibrate_channel_amax")


def sq_weight_channel_amax(layer: Layer, w, amax_k, stream=None) -> None:
    """Per-input-channel maxima of |w| over the output channels into amax_k (device fp32 [K])."""
    _check(load_library().sq_weight_channel_amax(C.byref(layer.c), _dptr(w), _dt(w), _dptr(amax_k), _stream(stream)),
           "sq_weight_channel_amax")


def sq_smooth_factors(layer: Layer, amax_x: np.ndarray, amax_w: np.ndarray, alpha) -> tuple:
    """Host computation: (smooth, smooth_inv) fp32 [K] from host arrays of channel maxima and one alpha per K-segment."""
    ax = np.ascontiguousarray(amax_x, dtype=np.float32)
    aw = np.ascontiguousarray(amax_w, dtype=np.float32)
    al = np.ascontiguousarray(alpha, dtype=np.float32)
    assert ax.shape == (layer.K,) and aw.shape == (layer.K,) and al.shape == (layer.S,)
    s, r = np.empty(layer.K, np.float32), np.empty(layer.K, np.float32)
    _check(load_library().sq_smooth_factors(C.byref(layer.c), ax.ctypes.data, aw.ctypes.data, al.ctypes.data, s.ctypes.data,
                                            r.ctypes.data), "sq_smooth_factors")
    return s, r


def sq_quantize_weight_smoothed(layer: Layer, w, smooth, wq, wscale, stream=None) -> None:
    """sq_quantize_weight of W diag(smooth); smooth: device fp32 [K]."""
    _check(load_library().sq_quantize_weight_smoothed(C.byref(layer.c), _dptr(w), _dt(w), _dptr(smooth), _dptr(wq),
                                                      _dptr(wscale), _stream(stream)), "sq_quantize_weight_smoothed")


def sq_quantize_act_smoothed(layer: Layer, x, smooth_inv, xq, stream=None) -> None:
    """sq_quantize_act of X diag(smooth_inv); smooth_inv: device fp32 [K]; the layer's steps are those of the smoothed X."""
    _check(load_library().sq_quantize_act_smoothed(C.byref(layer.c), _dptr(x), _dt(x), _dptr(smooth_inv), _dptr(xq),
                                                   _stream(stream)), "sq_quantize_act_smoothed")


def sq_lowrank_workspace_bytes(layer: Layer, rank: int) -> int:
    """Device bytes sq_lowrank_add needs as workspace for this layer and rank."""
    return int(load_library().sq_lowrank_workspace_bytes(C.byref(layer.c), int(rank)))


def sq_lowrank_add(layer: Layer, x, ld, lu, y_q, y, workspace, stream=None) -> None:
    """y = y_q + (x ld^T) lu^T: the 16-bit low-rank side branch (ld bf16 [rank][K], lu bf16 [N][rank], y_q fp32 or None)."""
    rank = int(ld.shape[0])
    _check(load_library().sq_lowrank_add(C.byref(layer.c), _dptr(x), _dt(x), _dptr(ld), _dptr(lu), rank, _dptr(y_q), _dptr(y),
                                         _dt(y), _dptr(workspace), workspace.numel() * workspace.element_size(),
                                         _stream(stream)), "sq_lowrank_add")


def sq_quantize_weight_fp8(layer: Layer, w, wq, wscale, stream=None) -> None:
    """w [N][K] fp32/bf16 -> wq uint8 [N][K] (E4M3 codes), wscale fp32 [S][N] = max|w| / 448 per channel and K-segment."""
    _check(load_library().sq_quantize_weight_fp8(C.byref(layer.c), _dptr(w), _dt(w), _dptr(wq), _dptr(wscale),
                                                 _stream(stream)), "sq_quantize_weight_fp8")


def sq_quantize_act_fp8(layer: Layer, x, xq, stream=None) -> None:
    """x [M][K] fp32/bf16 -> xq uint8 [M][K], E4M3 codes of Q_dual (X^_+: sign bit clear, X^_-: sign bit set)."""
    _check(load_library().sq_quantize_act_fp8(C.byref(layer.c), _dptr(x), _dt(x), _dptr(xq), _stream(stream)),
           "sq_quantize_act_fp8")


def sq_quantize_act_fp8_fused(layer: Layer, h, act, xq, workspace=None, stream=None) -> None:
    """xq = Q_dual(act(h)) with E4M3 codes: h [M][K] fp32/bf16 pre-activation, act: SQ_ACT_* per K-segment (host sequence);
    workspace: optional device byte tensor (checked, unused: the code tables of bf16 inputs live on chip)."""
    if len(act) != layer.c.S:
        raise ValueError("one activation code per K-segment")
    codes = (C.c_int32 * max(len(act), 1))(*[int(a) for a in act])
    nbytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    _check(load_library().sq_quantize_act_fp8_fused(C.byref(layer.c), _dptr(h), _dt(h), codes, _dptr(xq), _dptr(workspace),
                                                    nbytes, _stream(stream)), "sq_quantize_act_fp8_fused")


def sq_seglinear_fp8(layer: Layer, xq, wq, wscale, bias, y, stream=None) -> None:
    """The layer on fp8 codes: K-segment sums on the fp8 matrix cores (fp32 accumulation), dequantized into y."""
    _check(load_library().sq_seglinear_fp8(C.byref(layer.c), _dptr(xq), _dptr(wq), _dptr(wscale), _dptr(bias), _dptr(y),
                                           _dt(y), _stream(stream)), "sq_seglinear_fp8")


def sq_quantize_act(layer: Layer, x, xq, stream=None) -> None:
    """x [M][K] fp32/bf16 -> xq int8 [M][K], polarity-merged codes (X^_+ = max(xq, 0), X^_- = min(xq, 0))."""
    _check(load_library().sq_quantize_act(C.byref(layer.c), _dptr(x), _dt(x), _dptr(xq), _stream(stream)),
           "sq_quantize_act")


SQ_ACT_NONE, SQ_ACT_SILU, SQ_ACT_GELU = 0, 1, 2


def sq_quantize_act_fused_workspace_bytes(layer: Layer) -> int:
    """Device bytes that a workspace handed to sq_quantize_act_fused must have (64 KiB per K-segment)."""
    return int(load_library().sq_quantize_act_fused_workspace_bytes(C.byref(layer.c)))


def sq_quantize_act_fused(layer: Layer, h, act, xq, workspace=None, stream=None) -> None:
    """xq = Q_dual(act(h)): h [M][K] fp32/bf16 pre-activation, act: SQ_ACT_* per K-segment (host sequence);
    workspace: optional device byte tensor (checked, unused: the code tables of bf16 inputs live on chip)."""
    codes = (C.c_int32 * max(len(act), 1))(*[int(a) for a in act])
    if len(act) != layer.c.S:
        raise ValueError("one activation code per K-segment")
    nbytes = 0 if workspace is None else workspace.numel() * workspace.element_size()
    _check(load_library().sq_quantize_act_fused(C.byref(layer.c), _dptr(h), _dt(h), codes, _dptr(xq), _dptr(workspace),
                                                nbytes, _stream(stream)), "sq_quantize_act_fused")


def sq_unpack_w4(layer: Layer, wq4, wq, stream=None) -> None:
    """Packed 4-bit codes (sq_quantize_weight_w4) -> int8 [N][K], for the int8 GEMM entry points with the same wscale."""
    _check(load_library().sq_unpack_w4(C.byref(layer.c), _dptr(wq4), _dptr(wq), _stream(stream)), "sq_unpack_w4")


def sq_quantize_act_geglu(layer: Layer, h, xq, stream=None) -> None:
    """xq [M][K] = Q_dual(value * GELU(gate)): h [M][2K] fp32/bf16 = [value | gate]; the layer's K-segments are those of xq."""
    _check(load_library().sq_quantize_act_geglu(C.byref(layer.c), _dptr(h), _dt(h), _dptr(xq), _stream(stream)),
           "sq_quantize_act_geglu")


def sq_seglinear(layer: Layer, xq, wq, wscale, bias, y, stream=None) -> None:
    """int8 x int8 -> int32 per K-segment and polarity, dequantized into y [M][N] fp32/bf16."""
    _check(load_library().sq_seglinear(C.byref(layer.c), _dptr(xq), _dptr(wq), _dptr(wscale), _dptr(bias),
                                       _dptr(y), _dt(y), _stream(stream)), "sq_seglinear")


def sq_quantize_weight_w4(layer: Layer, w, wq4, wscale, stream=None) -> None:
    """w [N][K] fp32/bf16 -> wq4 uint8 [ceil(N/16)*16*K/2] (4-bit codes, two per byte, one KiB per 16-row group and
    128-code step), wscale fp32 [S][N]."""
    _check(load_library().sq_quantize_weight_w4(C.byref(layer.c), _dptr(w), _dt(w), _dptr(wq4), _dptr(wscale),
                                                _stream(stream)), "sq_quantize_weight_w4")


def sq_seglinear_w4(layer: Layer, xq, wq4, wscale, bias, y, stream=None) -> None:
    """sq_seglinear with 4-bit packed weights."""
    _check(load_library().sq_seglinear_w4(C.byref(layer.c), _dptr(xq), _dptr(wq4), _dptr(wscale), _dptr(bias),
                                          _dptr(y), _dt(y), _stream(stream)), "sq_seglinear_w4")


def sq_seglinear_w4_debug_acc(layer: Layer, xq, wq4, acc_pos, acc_neg, stream=None) -> None:
    """Raw int32 sums of the 4-bit codes: acc_pos, acc_neg int32 [S][M][N]."""
    _check(load_library().sq_seglinear_w4_debug_acc(C.byref(layer.c), _dptr(xq), _dptr(wq4), _dptr(acc_pos),
                                                    _dptr(acc_neg), _stream(stream)), "sq_seglinear_w4_debug_acc")


def sq_quantize_act_dynamic(layer: Layer, x, xq, tok_steps, stream=None) -> None:
    """Per-token min/max steps and codes: xq int8 [M][K], tok_steps fp32 [2][M][S] (s_pos, then s_neg)."""
    _check(load_library().sq_quantize_act_dynamic(C.byref(layer.c), _dptr(x), _dt(x), _dptr(xq), _dptr(tok_steps),
                                                  _stream(stream)), "sq_quantize_act_dynamic")


def sq_quantize_act_dynamic_bits(layer: Layer, x, a_bits: int, xq, tok_steps, stream=None) -> None:
    """sq_quantize_act_dynamic with a_bits-wide activation codes (8, or 4: codes in [-7, 7], one per byte)."""
    _check(load_library().sq_quantize_act_dynamic_bits(C.byref(layer.c), _dptr(x), _dt(x), int(a_bits), _dptr(xq),
                                                       _dptr(tok_steps), _stream(stream)), "sq_quantize_act_dynamic_bits")


def sq_seglinear_dynamic(layer: Layer, xq, tok_steps, wq, w_bits: int, wscale, bias, y, stream=None) -> None:
    """The layer with per-token steps; wq: int8 [N][K] (w_bits 8) or packed 4-bit codes (w_bits 4)."""
    _check(load_library().sq_seglinear_dynamic(C.byref(layer.c), _dptr(xq), _dptr(tok_steps), _dptr(wq), int(w_bits),
                                               _dptr(wscale), _dptr(bias), _dptr(y), _dt(y), _stream(stream)),
           "sq_seglinear_dynamic")


class GroupItems:
    """The marshalled item array of a grouped call (device pointers of L layers), built once and reused: filling
    it takes longer on the host than the launch takes on the GPU.  Keeps the tensors alive."""

    def __init__(self, items):
        self.tensors = list(items)
        self.n = len(self.tensors)
        self.arr = (sq_group_item * max(self.n, 1))()
        for i, (wq, wscale, bias, y) in enumerate(self.tensors):
            self.arr[i] = sq_group_item(wq.data_ptr(), wscale.data_ptr(), None if bias is None else bias.data_ptr(),
                                        y.data_ptr())
        self.y_dt = _dt(self.tensors[0][3]) if self.n else SQ_F32


def sq_seglinear_grouped(layer: Layer, xq, items, stream=None) -> None:
    """L layers of one shape sharing xq in one launch.  items: a GroupItems, or a sequence of (wq, wscale, bias or
    None, y) device tensors; all y of one dtype."""
    g = items if isinstance(items, GroupItems) else GroupItems(items)
    _check(load_library().sq_seglinear_grouped(C.byref(layer.c), _dptr(xq), g.n, g.arr, g.y_dt, _stream(stream)),
           "sq_seglinear_grouped")


def sq_seglinear_grouped_fp8(layer: Layer, xq, items, stream=None) -> None:
    """sq_seglinear_grouped on fp8 (E4M3) codes: xq and the items' wq are uint8 code tensors."""
    g = items if isinstance(items, GroupItems) else GroupItems(items)
    _check(load_library().sq_seglinear_grouped_fp8(C.byref(layer.c), _dptr(xq), g.n, g.arr, g.y_dt, _stream(stream)),
           "sq_seglinear_grouped_fp8")


def _act_codes(layer: Layer, act):
    if act is None:
        return None
    if len(act) != layer.c.S:
        raise ValueError("one activation code per K-segment")
    return (C.c_int32 * max(len(act), 1))(*[int(a) for a in act])


def sq_seglinear_fused(layer: Layer, x, act, wq, wscale, bias, y, stream=None) -> None:
    """y = SegLinear(Q_dual(act(x))) in one launch (skinny layers): x [M][K] fp32/bf16 raw activations, act: SQ_ACT_*
    per K-segment or None."""
    _check(load_library().sq_seglinear_fused(C.byref(layer.c), _dptr(x), _dt(x), _act_codes(layer, act), _dptr(wq),
                                             _dptr(wscale), _dptr(bias), _dptr(y), _dt(y), _stream(stream)),
           "sq_seglinear_fused")


def sq_seglinear_fused_dynamic(layer: Layer, x, act, wq, w_bits, wscale, bias, y, a_bits=8, stream=None) -> None:
    """sq_seglinear_fused with per-token activation steps found inside the launch; wq: int8 [N][K] (w_bits 8) or the packed
    4-bit codes of sq_quantize_weight_w4 (w_bits 4); a_bits: width of the activation codes (8 or 4)."""
    _check(load_library().sq_seglinear_fused_dynamic(C.byref(layer.c), _dptr(x), _dt(x), _act_codes(layer, act), int(a_bits),
                                                     _dptr(wq), int(w_bits), _dptr(wscale), _dptr(bias), _dptr(y), _dt(y),
                                                     _stream(stream)), "sq_seglinear_fused_dynamic")


def sq_seglinear_grouped_w4(layer: Layer, xq, items, tok_steps=None, stream=None) -> None:
    """sq_seglinear_grouped with packed 4-bit weights in the items (wq4 of sq_quantize_weight_w4); tok_steps: None for
    the layer's static steps, or the per-token steps [2][M][S] that belong to xq."""
    g = items if isinstance(items, GroupItems) else GroupItems(items)
    _check(load_library().sq_seglinear_grouped_w4(C.byref(layer.c), _dptr(xq), _dptr(tok_steps), g.n, g.arr, g.y_dt,
                                                  _stream(stream)), "sq_seglinear_grouped_w4")


def sq_seglinear_grouped_fused(layer: Layer, x, act, items, stream=None) -> None:
    """sq_seglinear_fused for L layers of one shape that share x; items as for sq_seglinear_grouped."""
    g = items if isinstance(items, GroupItems) else GroupItems(items)
    _check(load_library().sq_seglinear_grouped_fused(C.byref(layer.c), _dptr(x), _dt(x), _act_codes(layer, act), g.n,
                                                     g.arr, g.y_dt, _stream(stream)), "sq_seglinear_grouped_fused")


def sq_seglinear_debug_acc(layer: Layer, xq, wq, acc_pos, acc_neg, stream=None) -> None:
    """Same main loop, raw int32 accumulators: acc_pos, acc_neg int32 [S][M][N]."""
    _check(load_library().sq_seglinear_debug_acc(C.byref(layer.c), _dptr(xq), _dptr(wq), _dptr(acc_pos),
                                                 _dptr(acc_neg), _stream(stream)), "sq_seglinear_debug_acc")
