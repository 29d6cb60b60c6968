"""Python binding of the C ABI in include/splice_attn.h (ctypes).

Argument marshalling only: every step of the computation runs in the HIP
library.  Functions have the C names.  Tensor arguments are torch tensors
on the GPU; before calling into C the binding checks each tensor's device,
dtype, contiguity and element count against the shape, so that no call can
make a kernel read or write outside a buffer.  A negative status from C
raises SpliceError.  The library must be built
(``python -m paper_2605_30574_amd.build``); there is no fallback.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Sequence

import numpy as np

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libsplice_attn.so")

SPLICE_OK, SPLICE_EINVAL, SPLICE_ESHAPE, SPLICE_EWORKSPACE, SPLICE_EUNSUPPORTED, SPLICE_EHIP = 0, -1, -2, -3, -4, -5
SPLICE_DONOR_BUFFER, SPLICE_DONOR_ZERO = 0, 1
SPLICE_BF16, SPLICE_F32 = 0, 1
SPLICE_SRC_CLEAN, SPLICE_SRC_DONOR, SPLICE_SRC_ZERO, SPLICE_SRC_GEN = 0, 1, 2, 3
SPLICE_MAX_CELLS = 256
SPLICE_ABI_VERSION = 6   # layout of SpliceShape / SpliceCall below

EXPORTS = ("splice_abi_version", "splice_status_str", "splice_visible_len", "splice_kv_build",
           "splice_decode_attn_workspace_bytes", "splice_workspace_init", "splice_decode_attn",
           "splice_decode_step", "splice_decode_forked", "splice_workspace_handovers",
           "splice_decode_attn_noalloc")
SPLICE_NOALLOC_WORKSPACE_BYTES = 32 << 20


class SpliceShape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in (
        "n_cells", "n_layers", "n_q_heads", "n_kv_heads", "head_dim", "prompt_len",
        "span_lo", "span_hi", "gen_capacity", "donor_kind", "dtype")]


class SpliceCall(ctypes.Structure):
    _fields_ = [("layer", ctypes.c_int32), ("step", ctypes.c_int32), ("window", ctypes.c_int32),
                ("scale", ctypes.c_float), ("split_keys", ctypes.c_int32), ("merge_wait", ctypes.c_int32)]


class SpliceError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {status_name(status)} ({status})")


_lib = None
_torch = None                # torch, once the library is loaded
_current_raw_stream = None   # device index -> handle of its current stream, without a Stream object


def load_library(path: str = LIB_PATH):
    """Load libsplice_attn.so (after torch, so both share one HIP runtime)."""
    global _lib, _torch, _current_raw_stream
    if _lib is not None:
        return _lib
    import torch  # maps torch's libamdhip64 before ours resolves it
    _torch, _current_raw_stream = torch, getattr(torch._C, "_cuda_getCurrentRawStream", None)
    if not os.path.exists(path):
        raise ImportError(f"{path} is not built; run `python -m paper_2605_30574_amd.build`")
    lib = ctypes.CDLL(path)
    vp, i32 = ctypes.c_void_p, ctypes.c_int32
    shp, cal = ctypes.POINTER(SpliceShape), ctypes.POINTER(SpliceCall)
    i32p = vp   # host int32 arrays, by address
    lib.splice_abi_version.restype = i32
    lib.splice_abi_version.argtypes = []
    lib.splice_status_str.restype = ctypes.c_char_p
    lib.splice_status_str.argtypes = [i32]
    lib.splice_visible_len.restype = i32
    lib.splice_visible_len.argtypes = [shp, cal]
    lib.splice_kv_build.restype = i32
    lib.splice_kv_build.argtypes = [shp, cal, i32p, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.splice_decode_attn_workspace_bytes.restype = ctypes.c_int64
    lib.splice_decode_attn_workspace_bytes.argtypes = [shp, cal]
    lib.splice_workspace_init.restype = i32
    lib.splice_workspace_init.argtypes = [vp, ctypes.c_size_t, vp]
    lib.splice_workspace_handovers.restype = ctypes.c_int64
    lib.splice_workspace_handovers.argtypes = [vp, ctypes.c_size_t, vp]
    lib.splice_decode_attn.restype = i32
    lib.splice_decode_attn.argtypes = [shp, cal, i32p, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp,
                                       ctypes.c_size_t, vp]
    lib.splice_decode_attn_noalloc.restype = i32
    lib.splice_decode_attn_noalloc.argtypes = [shp, cal, i32p, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.splice_decode_step.restype = i32
    lib.splice_decode_step.argtypes = [shp, cal, i32p, i32p, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp,
                                       vp, ctypes.c_size_t, vp]
    lib.splice_decode_forked.restype = i32
    lib.splice_decode_forked.argtypes = [shp, cal, i32p, i32, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp,
                                         ctypes.c_size_t, vp]
    got = lib.splice_abi_version()
    if got != SPLICE_ABI_VERSION:
        raise ImportError(f"{path} has ABI version {got}, this binding expects {SPLICE_ABI_VERSION}: rebuild it")
    _lib = lib
    return lib


def status_name(status: int) -> str:
    try:
        return load_library().splice_status_str(int(status)).decode()
    except ImportError:
        return "unknown"


def _check(rc: int, where: str) -> int:
    if rc < 0:
        raise SpliceError(rc, where)
    return rc


# ------------------------------------------------------------------ helpers

def make_shape(n_cells: int, n_layers: int, n_q_heads: int, n_kv_heads: int, head_dim: int,
               prompt_len: int, span: Sequence[int], gen_capacity: int, donor_zero: bool,
               dtype: str) -> SpliceShape:
    return SpliceShape(n_cells, n_layers, n_q_heads, n_kv_heads, head_dim, prompt_len,
                       int(span[0]), int(span[1]), gen_capacity,
                       SPLICE_DONOR_ZERO if donor_zero else SPLICE_DONOR_BUFFER,
                       SPLICE_BF16 if dtype == "bf16" else SPLICE_F32)


def make_call(layer: int, step: int, window: int, scale: float, split_keys: int = 0,
              merge_wait: int = 0) -> SpliceCall:
    return SpliceCall(layer, step, window, float(scale), split_keys, merge_wait)


def _host_i32(x, rows: int, cols: int, name: str, what: str):
    """(array, address) of a contiguous host int32 array of rows x cols values; keep the array for the call."""
    if not (type(x) is np.ndarray and x.dtype == np.int32 and x.size == rows * cols and x.flags.c_contiguous):
        x = np.ascontiguousarray(np.asarray(x, dtype=np.int32).reshape((-1, cols) if cols > 1 else -1))
        if x.shape[0] != rows:
            raise ValueError(f"{name} has {x.shape[0]} {what}, shape says {rows} cells")
    return x, x.__array_interface__["data"][0]


def _cells(cell_LW, n_cells: int):
    return _host_i32(cell_LW, n_cells, 2, "cell_LW", "rows")


def _torch_dtype(shape: SpliceShape):
    return _torch.bfloat16 if shape.dtype == SPLICE_BF16 else _torch.float32


def _dev_ptr(t, name: str, numel: int, dtype, device=None, optional: bool = False):
    """Address of a contiguous GPU tensor of exactly ``numel`` elements, and its device."""
    if t is None:
        if optional:
            return None, device
        raise ValueError(f"{name} is required")
    if numel == 0 and t.numel() == 0:
        return None, (t.device if device is None else device)   # empty buffer: NULL
    if not t.is_cuda:
        raise ValueError(f"{name} must be a GPU tensor")
    if dtype is not None and t.dtype != dtype:
        raise ValueError(f"{name} has dtype {t.dtype}, expected {dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if numel is not None and t.numel() != numel:
        raise ValueError(f"{name} has {t.numel()} elements, expected {numel}")
    if device is not None and t.device != device:
        raise ValueError(f"{name} is on {t.device}, expected {device}")
    return t.data_ptr(), t.device


def _ptr(t, name: str, numel: int, dtype, dev):
    """_dev_ptr of a tensor on ``dev`` = (device index, device): the checks of the usual case in as few calls as they take
    (a call of the binding makes up to a dozen of them)."""
    if numel > 0 and t is not None and t.dtype is dtype and t.is_cuda and t.get_device() == dev[0] and \
            t.numel() == numel and t.is_contiguous():
        return t.data_ptr()
    return _dev_ptr(t, name, numel, dtype, dev[1])[0]


def _stream_ptr(stream, device):
    if stream is None:
        return _raw_stream(device)
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


def _raw_stream(device):
    """Handle of the current stream of ``device`` (a device, or its index)."""
    index = device if isinstance(device, int) else device.index
    if _current_raw_stream is not None and index is not None:
        return _current_raw_stream(index)
    return _torch.cuda.current_stream(device).cuda_stream


def _attn_ptrs(shape: SpliceShape, q, clean_k, clean_v, donor_k, donor_v, gen_k, gen_v, out, lse):
    """((device index, device), addresses) of the tensors every attention call takes, checked against the shape."""
    C, Hq, Hkv, D = shape.n_cells, shape.n_q_heads, shape.n_kv_heads, shape.head_dim
    dt = _torch_dtype(shape)
    n_prompt, n_gen, n_out = Hkv * shape.prompt_len * D, C * Hkv * shape.gen_capacity * D, C * Hq * D
    qp, device = _dev_ptr(q, "q", n_out, dt)
    dev = (q.get_device(), device)
    ck, cv = _ptr(clean_k, "clean_k", n_prompt, dt, dev), _ptr(clean_v, "clean_v", n_prompt, dt, dev)
    if shape.donor_kind == SPLICE_DONOR_ZERO:
        if donor_k is not None or donor_v is not None:
            raise ValueError("the ZERO donor takes no donor buffers")
        dk = dv = None
    else:
        dk, dv = _ptr(donor_k, "donor_k", n_prompt, dt, dev), _ptr(donor_v, "donor_v", n_prompt, dt, dev)
    f32 = _torch.float32
    return dev, (qp, ck, cv, dk, dv, _ptr(gen_k, "gen_k", n_gen, dt, dev), _ptr(gen_v, "gen_v", n_gen, dt, dev),
                 _ptr(out, "out", n_out, f32, dev), _ptr(lse, "lse", C * Hq, f32, dev))


# ------------------------------------------------------------------ C entry points

def splice_abi_version() -> int:
    return load_library().splice_abi_version()


def splice_status_str(status: int) -> str:
    return load_library().splice_status_str(int(status)).decode()


def splice_visible_len(shape: SpliceShape, call: SpliceCall) -> int:
    return _check(load_library().splice_visible_len(ctypes.byref(shape), ctypes.byref(call)),
                  "splice_visible_len")


def splice_decode_attn_workspace_bytes(shape: SpliceShape, call: Optional[SpliceCall] = None) -> int:
    lib = load_library()
    return _check(lib.splice_decode_attn_workspace_bytes(
        ctypes.byref(shape), ctypes.byref(call) if call is not None else None),
        "splice_decode_attn_workspace_bytes")


def splice_workspace_init(workspace, stream=None) -> None:
    lib = load_library()
    p, dev = _dev_ptr(workspace, "workspace", None, None)
    nbytes = workspace.numel() * workspace.element_size()
    _check(lib.splice_workspace_init(p, nbytes, _stream_ptr(stream, dev)), "splice_workspace_init")


def splice_workspace_handovers(workspace, stream=None) -> int:
    """Merges handed over since the workspace was initialised (synchronises ``stream``)."""
    lib = load_library()
    p, dev = _dev_ptr(workspace, "workspace", None, None)
    nbytes = workspace.numel() * workspace.element_size()
    return _check(lib.splice_workspace_handovers(p, nbytes, _stream_ptr(stream, dev)), "splice_workspace_handovers")


def new_workspace(shape: SpliceShape, call: Optional[SpliceCall] = None, device="cuda", stream=None):
    """Allocate (torch) and prepare a workspace for ``shape`` (and ``call``).

    Before it serves a shape with another number of (cell, KV head) pairs it is
    prepared again (``splice_workspace_init``)."""
    import torch
    nbytes = splice_decode_attn_workspace_bytes(shape, call)
    ws = torch.empty(max(256, (nbytes + 255) // 256 * 256), dtype=torch.uint8, device=device)
    splice_workspace_init(ws, stream)
    return ws


def splice_kv_build(shape: SpliceShape, call: SpliceCall, cell_LW, clean_k, clean_v, donor_k, donor_v,
                    gen_k, gen_v, out_k, out_v, out_src, stream=None) -> None:
    lib = load_library()
    C, Hkv, D = shape.n_cells, shape.n_kv_heads, shape.head_dim
    n_vis = splice_visible_len(shape, call)
    dt = _torch_dtype(shape)
    n_prompt = Hkv * shape.prompt_len * D
    ck, dev = _dev_ptr(clean_k, "clean_k", n_prompt, dt)
    cv, _ = _dev_ptr(clean_v, "clean_v", n_prompt, dt, dev)
    if shape.donor_kind == SPLICE_DONOR_ZERO:
        if donor_k is not None or donor_v is not None:
            raise ValueError("the ZERO donor takes no donor buffers")
        dk = dv = None
    else:
        dk, _ = _dev_ptr(donor_k, "donor_k", n_prompt, dt, dev)
        dv, _ = _dev_ptr(donor_v, "donor_v", n_prompt, dt, dev)
    gk, _ = _dev_ptr(gen_k, "gen_k", C * Hkv * shape.gen_capacity * D, dt, dev)
    gv, _ = _dev_ptr(gen_v, "gen_v", C * Hkv * shape.gen_capacity * D, dt, dev)
    ok, _ = _dev_ptr(out_k, "out_k", C * Hkv * n_vis * D, dt, dev)
    ov, _ = _dev_ptr(out_v, "out_v", C * Hkv * n_vis * D, dt, dev)
    os_, _ = _dev_ptr(out_src, "out_src", C * n_vis, _torch.uint8, dev)
    lw, lwp = _cells(cell_LW, C)
    _check(lib.splice_kv_build(ctypes.byref(shape), ctypes.byref(call), lwp, ck, cv, dk, dv, gk, gv,
                               ok, ov, os_, _stream_ptr(stream, dev)), "splice_kv_build")


def splice_decode_attn(shape: SpliceShape, call: SpliceCall, cell_LW, q, clean_k, clean_v, donor_k,
                       donor_v, gen_k, gen_v, out, lse, workspace, stream=None) -> None:
    lib = load_library()
    dev, ptrs = _attn_ptrs(shape, q, clean_k, clean_v, donor_k, donor_v, gen_k, gen_v, out, lse)
    wp, _ = _dev_ptr(workspace, "workspace", None, None, dev[1])
    wbytes = workspace.numel() * workspace.element_size()
    lw, lwp = _cells(cell_LW, shape.n_cells)
    _check(lib.splice_decode_attn(ctypes.byref(shape), ctypes.byref(call), lwp, *ptrs, wp, wbytes,
                                  _stream_ptr(stream, dev[1])), "splice_decode_attn")


def splice_decode_attn_noalloc(shape: SpliceShape, call: SpliceCall, cell_LW, q, clean_k, clean_v, donor_k,
                               donor_v, gen_k, gen_v, out, lse, stream=None) -> None:
    """splice_decode_attn with the library's own per-GPU workspace array
    (no workspace argument, nothing allocated)."""
    lib = load_library()
    dev, ptrs = _attn_ptrs(shape, q, clean_k, clean_v, donor_k, donor_v, gen_k, gen_v, out, lse)
    lw, lwp = _cells(cell_LW, shape.n_cells)
    _check(lib.splice_decode_attn_noalloc(ctypes.byref(shape), ctypes.byref(call), lwp, *ptrs,
                                          _stream_ptr(stream, dev[1])), "splice_decode_attn_noalloc")


def _steps(cell_step, n_cells: int):
    return _host_i32(cell_step, n_cells, 1, "cell_step", "entries")


def splice_decode_step(shape: SpliceShape, call: SpliceCall, cell_LW, cell_step, q, k_new, v_new, clean_k,
                       clean_v, donor_k, donor_v, gen_k, gen_v, out, lse, workspace, stream=None) -> None:
    """One decode pass with each cell at its own step ``cell_step[c]`` (< 0: finished).

    Appends ``k_new[c]``, ``v_new[c]`` ([C, Hkv, D]) as row ``cell_step[c]`` of the
    cell's generated caches, then attends as ``splice_decode_attn`` at that step.
    """
    lib = load_library()
    dev, ptrs = _attn_ptrs(shape, q, clean_k, clean_v, donor_k, donor_v, gen_k, gen_v, out, lse)
    C, n_new, dt = shape.n_cells, shape.n_cells * shape.n_kv_heads * shape.head_dim, _torch_dtype(shape)
    kn, vn = _ptr(k_new, "k_new", n_new, dt, dev), _ptr(v_new, "v_new", n_new, dt, dev)
    wp, _ = _dev_ptr(workspace, "workspace", None, None, dev[1])
    wbytes = workspace.numel() * workspace.element_size()
    lw, lwp = _cells(cell_LW, C)
    st, stp = _steps(cell_step, C)
    _check(lib.splice_decode_step(ctypes.byref(shape), ctypes.byref(call), lwp, stp, ptrs[0], kn, vn, *ptrs[1:], wp,
                                  wbytes, _stream_ptr(stream, dev[1])), "splice_decode_step")


def splice_decode_forked(shape: SpliceShape, call: SpliceCall, cell_LW, trunk: int, q, clean_k, clean_v,
                         donor_k, donor_v, gen_k, gen_v, out, lse, workspace, stream=None) -> None:
    """Attention of a forked sweep: cell ``trunk`` is the clean run; a cell that
    has diverged reads its generated rows below its onset W from the trunk, and
    a cell that has not takes the trunk's out and lse."""
    lib = load_library()
    dev, ptrs = _attn_ptrs(shape, q, clean_k, clean_v, donor_k, donor_v, gen_k, gen_v, out, lse)
    wp, _ = _dev_ptr(workspace, "workspace", None, None, dev[1])
    wbytes = workspace.numel() * workspace.element_size()
    lw, lwp = _cells(cell_LW, shape.n_cells)
    _check(lib.splice_decode_forked(ctypes.byref(shape), ctypes.byref(call), lwp, int(trunk), *ptrs, wp, wbytes,
                                    _stream_ptr(stream, dev[1])), "splice_decode_forked")
