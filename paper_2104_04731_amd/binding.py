"""Binding for include/conv2d_int8.h: same names, argument marshalling only.

The tensor-taking calls of a program's inner loop go through the extension module `_native` (csrc/py_native.cpp: checks,
result tensor, stream and library call in one native step; in Python they took 7 us of a 10-us call).  Size and
selection queries and the calls made once per layer use ctypes.  torch is used for device memory and streams, nothing
else.  There is no CPU fallback: if the HIP library has not been built, `load()` raises.
"""
from __future__ import annotations

import ctypes
import os

import torch

from . import build as _build

OK, ERR_INVALID_ARG, ERR_UNSUPPORTED, ERR_OVERFLOW_RISK, ERR_WORKSPACE, ERR_DEVICE = range(6)
LAYOUT_AUTO, LAYOUT_PACKED, LAYOUT_IM2COL, LAYOUT_PAD_ONLY, LAYOUT_IMPLICIT, LAYOUT_IMAGE_PACK = range(6)
TILE_BAND = -2   # CONV_TILE_BAND
TILE_STREAM = 256   # CONV_TILE_STREAM: the first of these tiles
TILE_PANEL = 512    # CONV_TILE_PANEL: query_stage's first one of conv2d_int8_panel
ENTRY_ONE_SHOT, ENTRY_EX, ENTRY_NHWC, ENTRY_DILATED, ENTRY_DILATED_DIRECT = range(5)
STAGE_STORED, STAGE_RESIDENT, STAGE_RESIDENT_RAW, STAGE_RESIDENT_REWRITE, STAGE_BAND, STAGE_AS_IS, STAGE_STREAM, STAGE_STREAM_REWRITE = range(8)
STAGE_NAMES = ("stored rewrites", "resident", "resident, raw weights", "resident, weights rewritten first", "band on NCHW", "as is", "streamed weights",
               "streamed weights, rewritten first")
LAYOUT_NAMES = {LAYOUT_AUTO: "auto", LAYOUT_PACKED: "packed", LAYOUT_IM2COL: "im2col",
                LAYOUT_PAD_ONLY: "pad_only", LAYOUT_IMPLICIT: "implicit",
                LAYOUT_IMAGE_PACK: "image_pack"}

EXPORTS = [
    "conv2d_int8", "conv2d_int8_static", "conv2d_int8_nhwc", "unpack_nhwc_int32", "requant_int8", "requant_pack_layout", "conv2d_int8_ex", "conv2d_int8_workspace_bytes", "conv2d_int8_packed",
    "conv2d_int8_query_tiling", "conv2d_int8_num_tiles", "conv2d_int8_tile_info",
    "conv2d_int8_tile_applies", "conv2d_int8_tile_lds_bytes", "pack_layout", "pack_layout_bytes", "pack_layout_nhwc",
    "pack_weights", "pack_weights_depth", "pack_weights_bytes", "im2col_int8", "im2col_bytes",
    "image_pack_desc", "image_pack_bytes", "image_pack_weights_bytes", "image_pack_int8", "image_pack_weights",
    "conv2d_int8_packed_requant", "conv2d_int8_packed_nhwc", "mfma_probe_int8", "im2col_nhwc_int8", "pack_weights_rsc",
    "dilated_desc", "dilation_pack_bytes", "dilation_pack_int8", "dilation_unpack_int32",
    "conv2d_int8_dilated_workspace_bytes", "conv2d_int8_dilated",
    "conv2d_int8_dilated_direct_workspace_bytes", "conv2d_int8_dilated_direct",
    "gemm_int8_nt", "select_layout", "select_layout_weighted", "layout_overheads",
    "conv_status_string", "conv2d_int8_resident", "conv2d_int8_resident_applies", "conv2d_int8_resident_tile_info",
    "conv2d_int8_query_stage", "conv2d_int8_stored", "conv2d_int8_resident_requant", "conv2d_int8_panel", "conv2d_int8_panel_workspace_bytes", "conv2d_int8_panel_tile_info",
]


class ConvDesc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("N", "C", "H", "W", "K", "R", "S", "stride", "pad")]


class ConvError(RuntimeError):
    def __init__(self, status, what):
        self.status = status
        super().__init__(f"{what}: {status_string(status)} ({status})")


_lib = None
_native = None


def _calls():
    """The native entry points (loads them on the first call; never builds, never falls back)."""
    global _native
    if _native is None:
        load()
        if not os.path.exists(_build.NATIVE):
            raise RuntimeError(f"{_build.NATIVE} is missing: run `python -m paper_2104_04731_amd.build` "
                               "(or __graft_entry__.build()) first")
        from . import _native as native
        native.set_error_class(ConvError)
        native.set_library(_lib._handle)
        _native = native
    return _native


def load(path: str | None = None):
    """Load the built library (never builds; never falls back)."""
    global _lib
    if _lib is not None:
        return _lib
    path = path or _build.LIB
    if not os.path.exists(path):
        raise RuntimeError(f"{path} is missing: run `python -m paper_2104_04731_amd.build` "
                           "(or __graft_entry__.build()) first")
    lib = ctypes.CDLL(path)
    i, vp, sz, dbl = ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_double
    dp, ip = ctypes.POINTER(ConvDesc), ctypes.POINTER(ctypes.c_int)
    sig = {
        "conv2d_int8": (i, [i] * 9 + [vp, vp, vp, vp]),
        "conv2d_int8_static": (i, [i] * 9 + [vp, vp, vp, vp]),
        "conv2d_int8_nhwc": (i, [i] * 9 + [vp, vp, vp, vp]),
        "unpack_nhwc_int32": (i, [i] * 4 + [vp, vp, vp]),
        "requant_int8": (i, [ctypes.c_longlong, vp, vp, i, i, vp]),
        "requant_pack_layout": (i, [i] * 8 + [vp, vp, vp]),
        "conv2d_int8_ex": (i, [dp, i, i, vp, vp, i, vp, vp, sz, vp]),
        "conv2d_int8_stored": (i, [dp, i, i, vp, vp, i, vp, vp, sz, vp]),
        "conv2d_int8_workspace_bytes": (sz, [dp, i, i, i]),
        "conv2d_int8_packed": (i, [dp, i, i, vp, vp, vp, i, i, vp]),
        "conv2d_int8_query_tiling": (i, [dp, i, i, ip, ip]),
        "conv2d_int8_tile_applies": (i, [dp, i, i, i, i]),
        "conv2d_int8_tile_lds_bytes": (sz, [dp, i, i, i, i]),
        "conv2d_int8_num_tiles": (i, []),
        "conv2d_int8_tile_info": (i, [i, ip, ip, ip, ip]),
        "pack_layout": (i, [i] * 6 + [vp, vp, vp]),
        "pack_layout_bytes": (sz, [i] * 6),
        "pack_layout_nhwc": (i, [i] * 6 + [vp, vp, vp]),
        "pack_weights": (i, [i] * 6 + [vp, vp, vp]),
        "pack_weights_depth": (i, [i] * 5),
        "pack_weights_bytes": (sz, [i] * 6),
        "im2col_int8": (i, [i] * 9 + [vp, vp, vp]),
        "im2col_bytes": (sz, [i] * 9),
        "im2col_nhwc_int8": (i, [i] * 9 + [vp, vp, vp]),
        "pack_weights_rsc": (i, [i] * 4 + [vp, vp, vp]),
        "image_pack_desc": (i, [dp, dp]),
        "image_pack_bytes": (sz, [dp]),
        "image_pack_weights_bytes": (sz, [dp]),
        "image_pack_int8": (i, [dp, vp, vp, vp]),
        "image_pack_weights": (i, [dp, vp, vp, vp]),
        "conv2d_int8_packed_requant": (i, [dp, i, i, vp, vp, vp, i, i, i, i, vp]),
        "conv2d_int8_resident_requant": (i, [dp, i, i, vp, vp, vp, i, i, i, i, i, i, vp]),
        "conv2d_int8_packed_nhwc": (i, [dp, i, i, vp, vp, vp, i, i, vp]),
        "dilated_desc": (i, [dp, i, dp]),
        "dilation_pack_bytes": (sz, [dp, i]),
        "dilation_pack_int8": (i, [dp, i, vp, vp, vp]),
        "dilation_unpack_int32": (i, [dp, i, vp, vp, vp]),
        "conv2d_int8_dilated_workspace_bytes": (sz, [dp, i, i, i]),
        "conv2d_int8_dilated": (i, [dp, i, i, i, vp, vp, vp, vp, sz, vp]),
        "mfma_probe_int8": (i, [i, i, vp, vp]),
        "conv2d_int8_dilated_direct_workspace_bytes": (sz, [dp, i, i]),
        "conv2d_int8_dilated_direct": (i, [dp, i, i, vp, vp, vp, vp, sz, vp]),
        "gemm_int8_nt": (i, [i, i, i, vp, vp, vp, vp]),
        "select_layout": (i, [dp, ip, ip, ctypes.POINTER(dbl)]),
        "select_layout_weighted": (i, [dp, dbl, dbl, ip, ip, ctypes.POINTER(dbl)]),
        "layout_overheads": (i, [dp, i, i] + [ctypes.POINTER(ctypes.c_int64)] * 3),
        "conv_status_string": (ctypes.c_char_p, [i]),
        "conv2d_int8_resident": (i, [dp, i, i, vp, vp, i, vp, i, i, vp]),
        "conv2d_int8_resident_applies": (i, [dp, i, i, i, i, i]),
        "conv2d_int8_resident_tile_info": (i, [i, ip, ip, ip]),
        "conv2d_int8_panel": (i, [dp, i, i, vp, vp, i, vp, i, i, vp, sz, vp]),
        "conv2d_int8_panel_workspace_bytes": (sz, [dp, i, i, i, i, i]),
        "conv2d_int8_panel_tile_info": (i, [i, ip, ip]),
        "conv2d_int8_query_stage": (i, [dp, i, i, i, i, i, ip, ip, ip]),
    }
    for name, (res, args) in sig.items():
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = res, args
    _lib = lib
    return lib


def status_string(status: int) -> str:
    return load().conv_status_string(int(status)).decode()


def _check(status, what):
    if status != OK:
        raise ConvError(status, what)


def _stream(stream=None):
    s = stream if stream is not None else torch.cuda.current_stream()
    return ctypes.c_void_p(s.cuda_stream)


def _ptr(t: torch.Tensor):
    return ctypes.c_void_p(t.data_ptr())


def _desc(N, C, H, W, K, R, S, stride, pad):
    return ConvDesc(N, C, H, W, K, R, S, stride, pad)


def out_hw(H, W, R, S, stride, pad):
    return (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1


def _require(t, dtype, what):
    if not (t.is_cuda and t.dtype == dtype and t.is_contiguous()):
        raise TypeError(f"{what} must be a contiguous {dtype} CUDA tensor")


# ---- one-shot -------------------------------------------------------------------------------
def conv2d_int8(x: torch.Tensor, w: torch.Tensor, stride: int, pad: int, out=None, stream=None):
    return (_native or _calls()).conv2d_int8(x, w, stride, pad, out, stream)


STATIC_WORKSPACE_BYTES = 8 << 20


def conv2d_int8_static(x: torch.Tensor, w: torch.Tensor, stride: int, pad: int, out: torch.Tensor, stream=None):
    """conv2d_int8 through the library's fixed device array: the call allocates nothing (`out` is the caller's)."""
    return (_native or _calls()).conv2d_int8_static(x, w, stride, pad, out, stream)


def conv2d_int8_nhwc(x: torch.Tensor, w: torch.Tensor, stride: int, pad: int, out=None, stream=None):
    """x: [N, H, W, C] int8, w: KCRS int8 -> [N, P, Q, K] int32."""
    return (_native or _calls()).conv2d_int8_nhwc(x, w, stride, pad, out, stream)


def unpack_nhwc_int32(x: torch.Tensor, out=None, stream=None):
    """[N, K, P, Q] int32 -> [N, P, Q, K] int32."""
    return (_native or _calls()).unpack_nhwc_int32(x, out, stream)


def requant_int8(x: torch.Tensor, shift: int, relu: bool, out=None, stream=None):
    """int32 tensor -> int8 tensor of the same shape: clip(relu(floor(x / 2^shift + 1/2)))."""
    return (_native or _calls()).requant_int8(x, shift, relu, out, stream)


def requant_pack_layout(x: torch.Tensor, cb: int, pad: int, shift: int, relu: bool, out=None, stream=None):
    """[N, K, P, Q] int32 -> [N, ceil(K/cb), P+2pad, Q+2pad, cb] int8: activation + the next layer's blocking."""
    return (_native or _calls()).requant_pack_layout(x, cb, pad, shift, relu, out, stream)


def conv2d_int8_workspace_bytes(dims, layout=LAYOUT_AUTO, cb=0, wt_is_packed=False) -> int:
    d = _desc(*dims)
    return int(load().conv2d_int8_workspace_bytes(ctypes.byref(d), layout, cb, int(wt_is_packed)))


def conv2d_int8_ex(dims, layout, cb, x, w, out, workspace, wt_is_packed=False, stream=None):
    return (_native or _calls()).conv2d_int8_ex(dims, layout, cb, x, w, out, workspace, wt_is_packed, stream)


def conv2d_int8_stored(dims, layout, cb, x, w, out, workspace, wt_is_packed=False, stream=None):
    """conv2d_int8_ex with the rewritten operands always stored in `layout`."""
    _check(load().conv2d_int8_stored(ctypes.byref(_desc(*dims)), layout, cb, _ptr(x), _ptr(w), int(wt_is_packed), _ptr(out),
                                     None if workspace is None else _ptr(workspace),
                                     0 if workspace is None else workspace.numel() * workspace.element_size(), _stream(stream)),
           "conv2d_int8_stored")
    return out


def conv2d_int8_packed(dims, layout, cb, x_packed, w_packed, out, tile=-1, split_k=0, stream=None):
    return (_native or _calls()).conv2d_int8_packed(dims, layout, cb, x_packed, w_packed, out, tile, split_k, stream)


def conv2d_int8_packed_nhwc(dims, layout, cb, x_packed, w_packed, out, tile=-1, split_k=0, stream=None):
    """GEMM stage writing int32 [N][P][Q][K]."""
    return (_native or _calls()).conv2d_int8_packed_nhwc(dims, layout, cb, x_packed, w_packed, out, tile, split_k, stream)


def tile_applies(dims, layout, cb, tile, split_k=1):
    """True if conv2d_int8_packed would accept this forced tile and depth split."""
    d = _desc(*dims)
    return load().conv2d_int8_tile_applies(ctypes.byref(d), layout, cb, tile, split_k) == OK


def tile_lds_bytes(dims, layout, cb, tile, split_k=1) -> int:
    d = _desc(*dims)
    return int(load().conv2d_int8_tile_lds_bytes(ctypes.byref(d), layout, cb, tile, split_k))


def query_tiling(dims, layout, cb):
    d = _desc(*dims)
    t, s = ctypes.c_int(), ctypes.c_int()
    _check(load().conv2d_int8_query_tiling(ctypes.byref(d), layout, cb, ctypes.byref(t), ctypes.byref(s)),
           "conv2d_int8_query_tiling")
    return t.value, s.value


def num_tiles() -> int:
    return load().conv2d_int8_num_tiles()


def tile_info(tile: int):
    r, c, t, k = ctypes.c_int(), ctypes.c_int(), ctypes.c_int(), ctypes.c_int()
    _check(load().conv2d_int8_tile_info(tile, ctypes.byref(r), ctypes.byref(c), ctypes.byref(t),
                                        ctypes.byref(k)), "conv2d_int8_tile_info")
    return r.value, c.value, t.value, k.value


# ---- GEMM stage on the network's own tensor ---------------------------------------------------
def conv2d_int8_resident(dims, x: torch.Tensor, w: torch.Tensor, out: torch.Tensor, wt_cb: int, tile: int, pixels: int, dilation=1, nhwc=False,
                         stream=None):
    """The stage that blocks the channels on its way into LDS, with this tile and pixels per workgroup (wt_cb 0: KCRS weights)."""
    _require(x, torch.int8, "input"); _require(w, torch.int8, "weights"); _require(out, torch.int32, "output")
    _check(load().conv2d_int8_resident(ctypes.byref(_desc(*dims)), dilation, int(nhwc), _ptr(x), _ptr(w), wt_cb, _ptr(out), tile, pixels,
                                       _stream(stream)), "conv2d_int8_resident")
    return out


def conv2d_int8_resident_requant(dims, layout, cb, x_packed: torch.Tensor, w_packed: torch.Tensor, out_cb, out_pad, shift, relu, out: torch.Tensor,
                                 tile: int, pixels: int, stream=None):
    """conv2d_int8_packed_requant through that stage, with this tile and pixels per workgroup (-1, 0: conv2d_int8_packed's stages)."""
    for t, what in ((x_packed, "input"), (w_packed, "weights"), (out, "output")):
        _require(t, torch.int8, what)
    _check(load().conv2d_int8_resident_requant(ctypes.byref(_desc(*dims)), layout, cb, _ptr(x_packed), _ptr(w_packed), _ptr(out), out_cb, out_pad, shift,
                                               int(relu), tile, pixels, _stream(stream)), "conv2d_int8_resident_requant")
    return out


def resident_applies(dims, wt_cb: int, tile: int, pixels: int, dilation=1, nhwc=False) -> bool:
    return load().conv2d_int8_resident_applies(ctypes.byref(_desc(*dims)), dilation, int(nhwc), wt_cb, tile, pixels) == OK


def resident_tiles():
    """(output channels, pixels of a wave, threads) of every tile."""
    out, v = [], [ctypes.c_int() for _ in range(3)]
    while load().conv2d_int8_resident_tile_info(len(out), *map(ctypes.byref, v)) == OK:
        out.append(tuple(x.value for x in v))
    return out


def stream_tiles():
    """{tile: (output channels, most pixels, threads)} of the tiles from TILE_STREAM on."""
    out, v = {}, [ctypes.c_int() for _ in range(3)]
    while load().conv2d_int8_resident_tile_info(TILE_STREAM + len(out), *map(ctypes.byref, v)) == OK:
        out[TILE_STREAM + len(out)] = tuple(x.value for x in v)
    return out


def conv2d_int8_panel(dims, x: torch.Tensor, w: torch.Tensor, out: torch.Tensor, wt_cb: int, tile: int, pixels: int, workspace: torch.Tensor,
                      dilation=1, nhwc=False, stream=None):
    """The stage that reads its weights in panels, with this tile and pixels per workgroup (wt_cb 0: KCRS weights)."""
    _require(x, torch.int8, "input"); _require(w, torch.int8, "weights"); _require(out, torch.int32, "output")
    _check(load().conv2d_int8_panel(ctypes.byref(_desc(*dims)), dilation, int(nhwc), _ptr(x), _ptr(w), wt_cb, _ptr(out), tile, pixels,
                                    _ptr(workspace), workspace.numel(), _stream(stream)), "conv2d_int8_panel")
    return out


def panel_workspace_bytes(dims, wt_cb: int, tile: int, pixels: int, dilation=1, nhwc=False) -> int:
    """0: the stage does not take this call."""
    return load().conv2d_int8_panel_workspace_bytes(ctypes.byref(_desc(*dims)), dilation, int(nhwc), wt_cb, tile, pixels)


def panel_tiles():
    """(output channels, most pixels) of every tile."""
    out, v = [], [ctypes.c_int() for _ in range(2)]
    while load().conv2d_int8_panel_tile_info(len(out), *map(ctypes.byref, v)) == OK:
        out.append(tuple(x.value for x in v))
    return out


def query_stage(dims, entry, layout=LAYOUT_AUTO, cb=0, wt_is_packed=False, dilation=1):
    """(stage, tile, pixels) of the call `entry` on tensors that start on 64 bytes."""
    v = [ctypes.c_int() for _ in range(3)]
    _check(load().conv2d_int8_query_stage(ctypes.byref(_desc(*dims)), entry, layout, cb, int(wt_is_packed), dilation, *map(ctypes.byref, v)),
           "conv2d_int8_query_stage")
    return tuple(x.value for x in v)


def stage_name(stage: int, tile: int, pixels: int) -> str:
    """query_stage's answer in words."""
    return "weights in panels" if stage == STAGE_STORED and tile >= TILE_PANEL else STAGE_NAMES[stage]


# ---- layout rewrites ------------------------------------------------------------------------
def pack_layout_bytes(N, C, H, W, cb, pad) -> int:
    return int(load().pack_layout_bytes(N, C, H, W, cb, pad))


def pack_layout(x: torch.Tensor, cb: int, pad: int, out=None, stream=None):
    return (_native or _calls()).pack_layout(x, cb, pad, out, stream)


def pack_layout_nhwc(x: torch.Tensor, cb: int, pad: int, out=None, stream=None):
    """x: [N, H, W, C] int8."""
    return (_native or _calls()).pack_layout_nhwc(x, cb, pad, out, stream)


def pack_weights_depth(C, R, S, layout, cb) -> int:
    return int(load().pack_weights_depth(C, R, S, layout, cb))


def pack_weights_bytes(K, C, R, S, layout, cb) -> int:
    return int(load().pack_weights_bytes(K, C, R, S, layout, cb))


def pack_weights(w: torch.Tensor, layout: int, cb: int, out=None, stream=None):
    return (_native or _calls()).pack_weights(w, layout, cb, out, stream)


def im2col_bytes(N, C, H, W, R, S, stride, pad, kg_pad) -> int:
    return int(load().im2col_bytes(N, C, H, W, R, S, stride, pad, kg_pad))


def im2col_int8(x: torch.Tensor, R, S, stride, pad, kg_pad=None, out=None, stream=None):
    return (_native or _calls()).im2col_int8(x, R, S, stride, pad, kg_pad, out, stream)


def im2col_nhwc_int8(xh: torch.Tensor, R, S, stride, pad, kg_pad=None, out=None, stream=None):
    """xh: [N, H, W, C] int8 -> [N*P*Q, kg_pad], depth index (r*S + s)*C + c."""
    return (_native or _calls()).im2col_nhwc_int8(xh, R, S, stride, pad, kg_pad, out, stream)


def pack_weights_rsc(w: torch.Tensor, out=None, stream=None):
    """KCRS int8 -> [K, ceil(C*R*S, 64)] in the depth order of im2col_nhwc_int8."""
    _require(w, torch.int8, "weights")
    K, C, R, S = w.shape
    if out is None:
        out = torch.empty((K, -(-C * R * S // 64) * 64), dtype=torch.int8, device=w.device)
    _check(load().pack_weights_rsc(K, C, R, S, _ptr(w), _ptr(out), _stream(stream)), "pack_weights_rsc")
    return out


def image_pack_desc(dims):
    """The stride-1, pad-0 problem (N, C2, H2, W2, K, R2, S2, 1, 0) an image-packed convolution turns into."""
    d, d2 = _desc(*dims), ConvDesc()
    _check(load().image_pack_desc(ctypes.byref(d), ctypes.byref(d2)), "image_pack_desc")
    return tuple(getattr(d2, f) for f, _ in ConvDesc._fields_)


def image_pack_int8(dims, x: torch.Tensor, out=None, stream=None):
    _require(x, torch.int8, "input")
    d = _desc(*dims)
    if out is None:
        N, C2, H2, W2 = image_pack_desc(dims)[:4]
        out = torch.empty((N, C2, H2, W2), dtype=torch.int8, device=x.device)
    _check(load().image_pack_int8(ctypes.byref(d), _ptr(x), _ptr(out), _stream(stream)), "image_pack_int8")
    return out


def image_pack_weights(dims, w: torch.Tensor, out=None, stream=None):
    _require(w, torch.int8, "weights")
    d = _desc(*dims)
    if out is None:
        _, C2, _, _, K, R2, S2, _, _ = image_pack_desc(dims)
        out = torch.empty((K, C2, R2, S2), dtype=torch.int8, device=w.device)
    _check(load().image_pack_weights(ctypes.byref(d), _ptr(w), _ptr(out), _stream(stream)), "image_pack_weights")
    return out


def conv2d_int8_packed_requant(dims, layout, cb, x_packed: torch.Tensor, w_packed: torch.Tensor, out_cb, out_pad, shift, relu,
                               out=None, stream=None):
    """GEMM stage with the activation in its epilogue: returns the next layer's blocked int8 input."""
    return (_native or _calls()).conv2d_int8_packed_requant(dims, layout, cb, x_packed, w_packed, out_cb, out_pad, shift, relu, out, stream)


def dilated_desc(dims, dilation):
    """The dense stride-1, pad-0 problem (N*d*d, C, H2, W2, K, R, S, 1, 0) a dilated convolution turns into."""
    d, d2 = _desc(*dims), ConvDesc()
    _check(load().dilated_desc(ctypes.byref(d), int(dilation), ctypes.byref(d2)), "dilated_desc")
    return tuple(getattr(d2, f) for f, _ in ConvDesc._fields_)


def dilated_out_hw(dims, dilation):
    N, C, H, W, K, R, S, stride, pad = dims
    return H + 2 * pad - dilation * (R - 1), W + 2 * pad - dilation * (S - 1)


def dilation_pack_int8(dims, dilation, x: torch.Tensor, out=None, stream=None):
    _require(x, torch.int8, "input")
    d = _desc(*dims)
    if out is None:
        N2, C, H2, W2 = dilated_desc(dims, dilation)[:4]
        out = torch.empty((N2, C, H2, W2), dtype=torch.int8, device=x.device)
    _check(load().dilation_pack_int8(ctypes.byref(d), int(dilation), _ptr(x), _ptr(out), _stream(stream)),
           "dilation_pack_int8")
    return out


def dilation_unpack_int32(dims, dilation, o2: torch.Tensor, out=None, stream=None):
    _require(o2, torch.int32, "sub-image results")
    d = _desc(*dims)
    if out is None:
        P, Q = dilated_out_hw(dims, dilation)
        out = torch.empty((dims[0], dims[4], P, Q), dtype=torch.int32, device=o2.device)
    _check(load().dilation_unpack_int32(ctypes.byref(d), int(dilation), _ptr(o2), _ptr(out), _stream(stream)),
           "dilation_unpack_int32")
    return out


def conv2d_int8_dilated_workspace_bytes(dims, dilation, layout=LAYOUT_AUTO, cb=0) -> int:
    return int(load().conv2d_int8_dilated_workspace_bytes(ctypes.byref(_desc(*dims)), int(dilation), int(layout), int(cb)))


def conv2d_int8_dilated(dims, dilation, x: torch.Tensor, w: torch.Tensor, layout=LAYOUT_AUTO, cb=0, out=None,
                        workspace=None, stream=None):
    """Stride-1 convolution with dilation >= 2: sub-images into the batch, dense convolution, interleave."""
    return (_native or _calls()).conv2d_int8_dilated(dims, dilation, x, w, layout, cb, out, workspace, stream)


def conv2d_int8_dilated_direct(dims, dilation, x: torch.Tensor, w: torch.Tensor, cb=0, out=None, workspace=None, stream=None):
    """Dilated convolution (any stride) with the dilation as an address multiplier of the GEMM stage."""
    return (_native or _calls()).conv2d_int8_dilated_direct(dims, dilation, x, w, 0, cb, out, workspace, stream)


def mfma_probe_int8(blocks: int, iters: int, out=None, stream=None, device="cuda:0"):
    """Register-resident MFMA loop; returns (checksums, operations issued)."""
    if out is None:
        out = torch.empty(blocks * 256, dtype=torch.int32, device=device)
    _check(load().mfma_probe_int8(int(blocks), int(iters), _ptr(out), _stream(stream)), "mfma_probe_int8")
    return out, 2 * 32768 * 16 * int(iters) * int(blocks)


def gemm_int8_nt(A: torch.Tensor, B: torch.Tensor, out=None, stream=None):
    return (_native or _calls()).gemm_int8_nt(A, B, out, stream)


# ---- selection (host only) --------------------------------------------------------------------
def select_layout(dims, w_mac=None, w_data=None):
    d = _desc(*dims)
    lay, cb, sc = ctypes.c_int(), ctypes.c_int(), ctypes.c_double()
    if w_mac is None:
        st = load().select_layout(ctypes.byref(d), ctypes.byref(lay), ctypes.byref(cb), ctypes.byref(sc))
    else:
        st = load().select_layout_weighted(ctypes.byref(d), w_mac, w_data, ctypes.byref(lay),
                                           ctypes.byref(cb), ctypes.byref(sc))
    _check(st, "select_layout")
    return lay.value, cb.value, sc.value


def layout_applies(dims, layout, cb=0) -> bool:
    """Whether the library has this layout for this problem (layout_overheads is the domain query)."""
    d = _desc(*dims)
    a, b, c = ctypes.c_int64(), ctypes.c_int64(), ctypes.c_int64()
    st = load().layout_overheads(ctypes.byref(d), layout, cb, ctypes.byref(a), ctypes.byref(b), ctypes.byref(c))
    if st not in (OK, ERR_UNSUPPORTED):
        raise ConvError(st, "layout_overheads")
    return st == OK


def layout_overheads(dims, layout, cb):
    d = _desc(*dims)
    a, b, c = ctypes.c_int64(), ctypes.c_int64(), ctypes.c_int64()
    _check(load().layout_overheads(ctypes.byref(d), layout, cb, ctypes.byref(a), ctypes.byref(b),
                                   ctypes.byref(c)), "layout_overheads")
    return a.value, b.value, c.value
