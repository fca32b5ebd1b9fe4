"""2-D CDF 9/7 and CDF 5/3 DWT on MI355X by non-separable lifting.

Thin binding over the C ABI of ``libdwt2.so`` (include/dwt2.h). Every step of
the transform runs in the library's HIP kernels; this module only checks
tensors, marshals pointers and picks the current HIP stream. PyTorch serves
for device memory and streams.

    import torch, paper_1705_08266_amd as dwt
    x = torch.rand(4096, 4096, device="cuda") * 255
    c = dwt.forward(x, "cdf97", levels=5)            # Mallat layout, same shape
    y = dwt.inverse(c, "cdf97", levels=5)
"""
from __future__ import annotations

import ctypes

from . import _lib
from ._lib import DWT2Error, load  # noqa: F401

WAVELETS = {"cdf97": _lib.CDF97, "cdf53": _lib.CDF53}
SCHEMES = {"nonseparable": _lib.NONSEPARABLE, "separable": _lib.SEPARABLE,
           # every neighbour exchange through LDS: the barrier-count ablation
           "nonseparable_lds": _lib.NONSEPARABLE_LDS, "separable_lds": _lib.SEPARABLE_LDS}


# Calls on small images cost what the host does per call (a 64 x 64 forward with
# three levels: 13.9 us, of which 3.8 in the library, against 7.9 on the device),
# so the marshalling below looks things up once: the torch module, descriptors
# and workspace sizes by their values, and the stream as the raw handle
# (torch.cuda.current_stream() builds an object: 2.7 us).
_torch_module = None
_DTYPE_CODES = {}
_CACHE_MAX = 256             # entries of each cache below
_descs = {}                  # (width, height, pitch, dtype code) -> pointer to its dwt2_desc
_workspace_floats = {}       # (width, height, levels) -> floats


def _torch():
    global _torch_module
    if _torch_module is None:
        import torch
        _DTYPE_CODES.update({torch.float32: _lib.F32, torch.float16: _lib.F16,
                             torch.bfloat16: _lib.BF16})
        _torch_module = torch
    return _torch_module


def _dtype_code(t) -> int:
    if _torch_module is None:
        _torch()
    code = _DTYPE_CODES.get(t.dtype)
    if code is None:
        raise TypeError(f"unsupported dtype {t.dtype}; use float32, float16 or bfloat16")
    return code


def _check_2d(t, name):
    if not t.is_cuda:
        raise ValueError(f"{name} must be a GPU tensor")
    if t.dim() != 2 or t.stride(1) != 1:
        raise ValueError(f"{name} must be 2-D with unit stride along rows")


def _desc(t):
    """Pointer to the dwt2_desc of a 2-D tensor (only ever read by the library)."""
    h, w = t.shape
    key = (w, h, t.stride(0), _dtype_code(t))
    d = _descs.get(key)
    if d is None:
        if len(_descs) >= _CACHE_MAX:
            _descs.clear()
        d = _descs[key] = ctypes.byref(_lib.Desc(*key))
    return d


def _wavelet(w) -> int:
    return WAVELETS[w] if isinstance(w, str) else int(w)


def _scheme(s) -> int:
    return SCHEMES[s] if isinstance(s, str) else int(s)


def _stream_ptr(stream=None) -> int:
    if stream is not None:
        return stream.cuda_stream
    torch = _torch()
    return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())


def _tiles_arg(tiles, levels):
    if tiles is None:
        return None
    if len(tiles) != levels:
        raise ValueError("need one tile id per level")
    return (ctypes.c_int32 * levels)(*[int(t) for t in tiles])


def _events_arg(events, levels):
    if events is None:
        return None
    if len(events) != 2 * levels:
        raise ValueError("need two events per level")
    for e in events:
        if not e.cuda_event:     # PyTorch creates the HIP event on its first record
            e.record()
    return (ctypes.c_void_p * (2 * levels))(*[e.cuda_event for e in events])


def workspace_bytes(width: int, height: int, levels: int, dtype=_lib.F32) -> int:
    """Workspace bytes of an L-level transform (the same for every storage
    type: intermediate low-low bands are FP32)."""
    return int(load().dwt2_workspace_bytes(width, height, levels, int(dtype)))


def _workspace_size(width: int, height: int, levels) -> int:
    """Floats of workspace, looked up by value; levels that are no plain int
    (anything ctypes takes for one, a tensor or an array among them) are asked
    for each time."""
    if type(levels) is not int:
        return workspace_bytes(width, height, levels) // 4
    key = (width, height, levels)
    n = _workspace_floats.get(key)
    if n is None:
        if len(_workspace_floats) >= _CACHE_MAX:
            _workspace_floats.clear()
        n = _workspace_floats[key] = workspace_bytes(*key) // 4
    return n


def make_workspace(width: int, height: int, levels: int, device=None):
    torch = _torch()
    n = workspace_bytes(width, height, levels)
    return torch.empty(max(1, n // 4), dtype=torch.float32, device=device or "cuda")


def _transform(plain, hooked, src, name, wavelet, levels, scheme, out, workspace, tiles, events,
               stream):
    torch = _torch()
    _check_2d(src, name)
    if out is None:
        out = torch.empty_like(src)
    _check_2d(out, "out")
    if workspace is None:
        n = _workspace_size(src.shape[1], src.shape[0], levels)
        if n:
            workspace = torch.empty(n, dtype=torch.float32, device=src.device)
    if workspace is not None:
        ws_ptr, ws_n = workspace.data_ptr(), workspace.numel() * workspace.element_size()
    else:
        ws_ptr, ws_n = None, 0
    lib = load()
    if tiles is None and events is None:
        st = getattr(lib, plain)(src.data_ptr(), _desc(src), out.data_ptr(), _desc(out),
                                 _wavelet(wavelet), levels, _lib.EXT_WHOLE_SAMPLE_SYMMETRIC,
                                 _scheme(scheme), ws_ptr, ws_n, _stream_ptr(stream))
    else:
        st = getattr(lib, hooked)(src.data_ptr(), _desc(src), out.data_ptr(), _desc(out),
                                  _wavelet(wavelet), levels, _lib.EXT_WHOLE_SAMPLE_SYMMETRIC,
                                  _scheme(scheme), ws_ptr, ws_n, _tiles_arg(tiles, levels),
                                  _events_arg(events, levels), _stream_ptr(stream))
    if st:
        _lib.check(st, plain)
    return out


def forward(x, wavelet="cdf97", levels: int = 1, scheme="nonseparable", out=None,
            workspace=None, tiles=None, events=None, stream=None):
    """L-level forward DWT of a 2-D GPU image; returns the Mallat-layout
    coefficients (same shape and dtype)."""
    return _transform("dwt2_forward", "dwt2_forward_ex", x, "x", wavelet, levels, scheme, out,
                      workspace, tiles, events, stream)


def forward_no_alloc(x, out, wavelet="cdf97", levels: int = 1, scheme="nonseparable",
                     stream=None):
    """:func:`forward` into a caller-provided `out`, with the library's own
    device workspace: the call allocates nothing (for graph capture and
    allocation-free loops). Calls on one GPU share that workspace and must not
    overlap in time."""
    _check_2d(x, "x")
    _check_2d(out, "out")
    st = load().dwt2_forward_no_alloc(x.data_ptr(), _desc(x), out.data_ptr(), _desc(out),
                                      _wavelet(wavelet), levels,
                                      _lib.EXT_WHOLE_SAMPLE_SYMMETRIC, _scheme(scheme),
                                      _stream_ptr(stream))
    _lib.check(st, "dwt2_forward_no_alloc")
    return out


def inverse(c, wavelet="cdf97", levels: int = 1, scheme="nonseparable", out=None,
            workspace=None, tiles=None, events=None, stream=None):
    """Inverse of :func:`forward`."""
    return _transform("dwt2_inverse", "dwt2_inverse_ex", c, "c", wavelet, levels, scheme, out,
                      workspace, tiles, events, stream)


def forward_level(x, ll, hl, lh, hh, wavelet="cdf97", scheme="nonseparable", tile=-1,
                  stream=None):
    """One level: x (H x W) -> four (H/2 x W/2) bands. hl, lh and hh must share
    one row pitch (e.g. views into a Mallat array)."""
    for t, n in ((x, "x"), (ll, "ll"), (hl, "hl"), (lh, "lh"), (hh, "hh")):
        _check_2d(t, n)
    if not (hl.stride(0) == lh.stride(0) == hh.stride(0)):
        raise ValueError("hl, lh and hh must share a row pitch")
    H, W = x.shape
    st = load().dwt2_forward_level(
        x.data_ptr(), x.stride(0), _dtype_code(x), W, H,
        ll.data_ptr(), ll.stride(0), _dtype_code(ll),
        hl.data_ptr(), lh.data_ptr(), hh.data_ptr(), hl.stride(0), _dtype_code(hl),
        _wavelet(wavelet), _scheme(scheme), int(tile), _stream_ptr(stream))
    _lib.check(st, "dwt2_forward_level")


def inverse_level(ll, hl, lh, hh, out, wavelet="cdf97", scheme="nonseparable", tile=-1,
                  stream=None):
    for t, n in ((out, "out"), (ll, "ll"), (hl, "hl"), (lh, "lh"), (hh, "hh")):
        _check_2d(t, n)
    if not (hl.stride(0) == lh.stride(0) == hh.stride(0)):
        raise ValueError("hl, lh and hh must share a row pitch")
    H, W = out.shape
    st = load().dwt2_inverse_level(
        ll.data_ptr(), ll.stride(0), _dtype_code(ll),
        hl.data_ptr(), lh.data_ptr(), hh.data_ptr(), hl.stride(0), _dtype_code(hl),
        out.data_ptr(), out.stride(0), _dtype_code(out), W, H,
        _wavelet(wavelet), _scheme(scheme), int(tile), _stream_ptr(stream))
    _lib.check(st, "dwt2_inverse_level")


def tile_configs(wavelet="cdf97"):
    """[(id, quads_per_lane, rows, waves, out_x, out_y)] compiled in."""
    lib = load()
    out = []
    for t in range(lib.dwt2_tile_config_count()):
        v = [ctypes.c_int32() for _ in range(5)]
        _lib.check(lib.dwt2_tile_config_info(t, _wavelet(wavelet), *[ctypes.byref(a) for a in v]))
        out.append((t, *[a.value for a in v]))
    return out


def fused_levels(width: int, height: int, levels: int) -> int:
    """Trailing levels the library runs as one fused launch by default."""
    n = int(load().dwt2_fused_levels(width, height, levels))
    _lib.check(min(n, 0), "dwt2_fused_levels")
    return n


def head_levels(width: int, height: int, levels: int) -> int:
    """Leading levels (0 or 2) the library runs as one fused launch by default."""
    n = int(load().dwt2_head_levels(width, height, levels))
    _lib.check(min(n, 0), "dwt2_head_levels")
    return n


def head_layout(src, dst, wavelet="cdf97", levels: int = 2, inverse=False):
    """(rows, tasks, streamed) of a fused head of levels 1 and 2 of
    forward(src, out=dst) or inverse(src, out=dst): rows of level 2 to a segment
    of its strips (0: it runs by windows), strips times segments (or windows),
    and whether its results are stored past the caches."""
    v = [ctypes.c_int32() for _ in range(3)]
    _lib.check(load().dwt2_head_layout(src.data_ptr(), _desc(src), dst.data_ptr(), _desc(dst),
                                       _wavelet(wavelet), levels, int(bool(inverse)),
                                       *[ctypes.byref(a) for a in v]), "dwt2_head_layout")
    return v[0].value, v[1].value, bool(v[2].value)


def default_tile(width, height, wavelet="cdf97", scheme="nonseparable", dtype=_lib.F32):
    return int(load().dwt2_default_tile(width, height, _wavelet(wavelet), _scheme(scheme), dtype))
