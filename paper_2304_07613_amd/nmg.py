"""ctypes binding of ``libnmg.so`` (declared in ``include/nmg.h``).

Argument marshalling only: torch allocates the outputs on the input's device
and supplies the current HIP stream; every step of the computation runs in the
library's HIP kernels.  There is no fallback: if the library is missing or a
call fails, the binding raises.

Paper: STen (arXiv 2304.07613), Section 5 (n:m:g layout), 5.1 (sparse x dense
product), 5.2 (magnitude converter and conversion back to dense).
"""
from __future__ import annotations

import ctypes
import os
import re

import torch

from . import build as _build

LIB_PATH = _build.LIB_PATH

F32, F16 = 0, 1
_DTYPE_CODE = {torch.float32: F32, torch.float16: F16}
KERNELS = {"auto": 0, "valu": 1, "mfma": 2, "mfma_general": 3, "mfma_scalar": 4, "mfma_f16": 5,
           "mfma_direct": 6, "smfmac_f16": 7, "valu_staged": 8, "mfma_wide": 9, "mfma_split": 10,
           "mfma_expand": 11, "sparse": 12}
_KERNEL_NAME = {v: k for k, v in KERNELS.items()}
EPILOGUES = {"none": 0, "gelu": 1, "add": 2}

OK, ERR_NULL, ERR_PARAM, ERR_SHAPE, ERR_DTYPE, ERR_ALIGN, ERR_LAUNCH, ERR_UNSUPPORTED, ERR_CAPACITY = \
    range(9)


class NmgError(RuntimeError):
    """A libnmg call returned a status other than NMG_OK."""

    def __init__(self, status: int, what: str):
        super().__init__(f"{what}: {status_str(status)} (status {status})")
        self.status = status


class _Layout(ctypes.Structure):
    _fields_ = [("M", ctypes.c_int32), ("K", ctypes.c_int32), ("n", ctypes.c_int32),
                ("m", ctypes.c_int32), ("g", ctypes.c_int32), ("C", ctypes.c_int32),
                ("dtype", ctypes.c_int)]


class _PLayout(ctypes.Structure):
    _fields_ = [("M", ctypes.c_int32), ("K", ctypes.c_int32), ("n", ctypes.c_int32),
                ("m", ctypes.c_int32), ("g", ctypes.c_int32), ("P", ctypes.c_int32),
                ("S", ctypes.c_int32), ("B", ctypes.c_int32), ("dtype", ctypes.c_int)]


_lib = None


def header_functions() -> list:
    """Names of the functions ``include/nmg.h`` declares."""
    with open(_build.HEADER) as f:
        text = f.read()
    return sorted(set(re.findall(r"^[A-Za-z_][\w \t\*]*?\b(nmg_\w+)\s*\(", text, re.M)))


def lib():
    """The loaded library; raises if it has not been built."""
    return _lib if _lib is not None else _load()


def _load():
    global _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} is not built; run __graft_entry__.build()")
    L = ctypes.CDLL(LIB_PATH)
    vp, i64, i32, lp = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.POINTER(_Layout)
    pp = ctypes.POINTER(_PLayout)
    sig = {
        "nmg_layout_init": ([lp, i32, i32, i32, i32, i32, ctypes.c_int], ctypes.c_int),
        "nmg_values_numel": ([lp], i64),
        "nmg_indices_numel": ([lp], i64),
        "nmg_compress": ([lp, vp, i64, vp, vp, vp], ctypes.c_int),
        "nmg_repack": ([lp, vp, i64, vp, vp, vp], ctypes.c_int),
        "nmg_spmm": ([lp, vp, vp, vp, i64, i64, vp, i64, vp], ctypes.c_int),
        "nmg_spmm_with": ([lp, ctypes.c_int, vp, vp, vp, i64, i64, vp, i64, vp], ctypes.c_int),
        "nmg_spmm_epilogue": ([lp, ctypes.c_int, ctypes.c_int, vp, vp, vp, i64, i64, vp, i64, vp,
                               i64, vp], ctypes.c_int),
        "nmg_spmm_epilogue_noalloc": ([lp, ctypes.c_int, ctypes.c_int, vp, vp, vp, i64, i64, vp,
                                       i64, vp, i64, vp], ctypes.c_int),
        "nmg_spmm_epilogue_ws": ([lp, ctypes.c_int, ctypes.c_int, vp, vp, vp, i64, i64, vp, i64, vp,
                                  i64, vp, i64, vp], ctypes.c_int),
        "nmg_spmm_workspace_bytes": ([lp, ctypes.c_int, i64], i64),
        "nmg_spmm_plan": ([lp, ctypes.c_int, vp, vp, vp, i64, i64, ctypes.POINTER(i64)],
                          ctypes.c_int),
        "nmg_p_spmm_ws": ([pp, ctypes.c_int, vp, vp, vp, i64, i64, vp, i64, vp, i64, vp],
                          ctypes.c_int),
        "nmg_p_spmm_workspace_bytes": ([pp, ctypes.c_int, i64], i64),
        "nmg_spmm_auto_kernel": ([lp, i64], ctypes.c_int),
        "nmg_densify": ([lp, vp, vp, vp, i64, vp], ctypes.c_int),
        "nmg_gelu": ([ctypes.c_int, vp, vp, i64, vp], ctypes.c_int),
        "nmg_add": ([ctypes.c_int, vp, vp, vp, i64, vp], ctypes.c_int),
        "nmg_p_layout_init": ([pp, i32, i32, i32, i32, i32, ctypes.c_int], ctypes.c_int),
        "nmg_p_compress": ([pp, vp, i64, vp, vp, vp], ctypes.c_int),
        "nmg_p_spmm": ([pp, vp, vp, vp, i64, i64, vp, i64, vp], ctypes.c_int),
        "nmg_p_spmm_with": ([pp, ctypes.c_int, vp, vp, vp, i64, i64, vp, i64, vp], ctypes.c_int),
        "nmg_p_refine": ([pp, vp, i64, vp, vp, vp], ctypes.c_int),
        "nmg_p_densify": ([pp, vp, vp, vp, i64, vp], ctypes.c_int),
        "nmg_x16_prepared_bytes": ([lp], i64),
        "nmg_x16_prepare": ([lp, vp, vp, vp, vp], ctypes.c_int),
        "nmg_spmm_x16": ([lp, vp, vp, i64, i64, vp, i64, vp], ctypes.c_int),
        "nmg_spmm_x16_epilogue": ([lp, vp, ctypes.c_int, vp, i64, i64, vp, i64, vp, i64, vp],
                                  ctypes.c_int),
        "nmg_status_str": ([ctypes.c_int], ctypes.c_char_p),
        "nmg_version": ([], ctypes.c_char_p),
    }
    for name, (args, res) in sig.items():
        fn = getattr(L, name)
        fn.argtypes = args
        fn.restype = res
    _lib = L
    return L


def status_str(status: int) -> str:
    return lib().nmg_status_str(status).decode()


def version() -> str:
    return lib().nmg_version().decode()


def _check(status: int, what: str):
    if status != OK:
        raise NmgError(status, what)


class Layout:
    """Shape of one n:m:g weight (``nmg_layout``)."""

    def __init__(self, M: int, K: int, n: int, m: int, g: int, dtype=torch.float32):
        if dtype not in _DTYPE_CODE:
            raise TypeError(f"unsupported dtype {dtype}")
        self.c = _Layout()
        _check(lib().nmg_layout_init(ctypes.byref(self.c), M, K, n, m, g, _DTYPE_CODE[dtype]),
               "nmg_layout_init")
        self.dtype = dtype
        self._derive()

    def _derive(self):
        c = self.c
        self.M, self.K, self.n, self.m, self.g, self.C = c.M, c.K, c.n, c.m, c.g, c.C
        self.values_shape = (self.M, self.C * self.n)
        self.indices_shape = (self.M // self.g, self.C * self.n)
        self._ws = (None, 0)     # what sized the last product's workspace, and its bytes

    def __setstate__(self, state):     # (also states of c and dtype alone)
        self.__dict__.update(state)
        self._derive()

    def __repr__(self):
        return (f"Layout(M={self.M}, K={self.K}, n={self.n}, m={self.m}, g={self.g}, "
                f"C={self.C}, dtype={self.dtype})")


def _stream(t: torch.Tensor) -> int:
    """The raw handle of the current stream of t's device."""
    return torch._C._cuda_getCurrentRawStream(t.get_device())


def _need_cuda(*ts):
    """Every tensor on the current GPU: the library launches on the current
    HIP device, on that device's current stream."""
    cur = -1
    for t in ts:
        dev = t.get_device()
        if dev < 0 or not t.is_cuda:
            raise ValueError("libnmg works on GPU tensors only")
        if cur < 0:
            cur = torch._C._cuda_getDevice()
        if dev != cur:
            raise ValueError(f"tensor on {t.device}, but the current device is cuda:{cur} "
                             "(select it with torch.cuda.device)")


def _rows(t: torch.Tensor, name: str) -> int:
    """Leading dimension of a 2-D row-major tensor (unit stride along rows)."""
    st = t.stride()
    if len(st) != 2 or st[1] != 1:
        raise ValueError(f"{name} must be a 2-D tensor with unit column stride")
    return st[0]


def _packed_ok(layout, values, indices):
    if values.shape != layout.values_shape or not values.is_contiguous():
        raise ValueError(f"values must be contiguous {layout.values_shape}")
    if indices.shape != layout.indices_shape or not indices.is_contiguous():
        raise ValueError(f"indices must be contiguous {layout.indices_shape}")


def _workspace(nbytes: int, like: torch.Tensor):
    """Scratch memory of one call from torch's allocator: (tensor, pointer,
    bytes).  Freed after the call returns; the allocator hands it out again in
    stream order on the current stream only.  None when the memory is not there:
    the library then takes what it takes without a workspace."""
    if nbytes <= 0:
        return None, None, 0
    try:
        ws = torch.empty(nbytes, dtype=torch.uint8, device=like.device)
    except torch.OutOfMemoryError:
        return None, None, 0
    return ws, ws.data_ptr(), nbytes


def _workspace_bytes(layout, code: int, vp: int, ip: int, xp: int, ldx: int, N: int) -> int:
    """The workspace of nmg_spmm_plan: a function of the layout, kernel, sizes and
    the pointers' alignment to 16 bytes."""
    at = (code, N, ldx, vp & 15, ip & 15, xp & 15)
    key, nbytes = layout._ws
    if key != at:
        out = ctypes.c_int64(0)
        lib().nmg_spmm_plan(layout.c, code, vp, ip, xp, ldx, N, ctypes.byref(out))
        nbytes = out.value
        layout._ws = (at, nbytes)
    return nbytes


def compress_into(layout: Layout, W: torch.Tensor, values: torch.Tensor, indices: torch.Tensor):
    """``nmg_compress`` into caller-allocated ``values`` / ``indices``."""
    _need_cuda(W, values, indices)
    if W.dtype != layout.dtype or values.dtype != layout.dtype or indices.dtype != torch.uint8:
        raise TypeError("dtype mismatch")
    if W.shape != (layout.M, layout.K):
        raise ValueError(f"W must be {layout.M} x {layout.K}")
    _packed_ok(layout, values, indices)
    _check(lib().nmg_compress(layout.c, W.data_ptr(), _rows(W, "W"), values.data_ptr(),
                              indices.data_ptr(), _stream(W)), "nmg_compress")


def compress(W: torch.Tensor, n: int, m: int, g: int):
    """Dense W (M x K, GPU) -> (values, indices, layout)."""
    layout = Layout(W.shape[0], W.shape[1], n, m, g, W.dtype)
    values = W.new_empty(layout.values_shape)
    indices = torch.empty(layout.indices_shape, dtype=torch.uint8, device=W.device)
    compress_into(layout, W, values, indices)
    return values, indices, layout


def repack(W: torch.Tensor, indices: torch.Tensor, layout: Layout) -> torch.Tensor:
    """Dense W (M x K, GPU) packed into the existing pattern `indices`
    (the fixed-mask path after a weight update) -> values."""
    _need_cuda(W, indices)
    if W.dtype != layout.dtype or indices.dtype != torch.uint8:
        raise TypeError("dtype mismatch")
    if W.shape != (layout.M, layout.K):
        raise ValueError(f"W must be {layout.M} x {layout.K}")
    if indices.shape != layout.indices_shape or not indices.is_contiguous():
        raise ValueError(f"indices must be contiguous {layout.indices_shape}")
    values = W.new_empty(layout.values_shape)
    _check(lib().nmg_repack(layout.c, W.data_ptr(), _rows(W, "W"), indices.data_ptr(),
                            values.data_ptr(), _stream(W)), "nmg_repack")
    return values


# kernel families that run on prepared operands (made per call by
# nmg_spmm_with, or once by nmg_x16_prepare for nmg_spmm_x16), and the element
# type each takes
X16_KERNELS = {"mfma_wide": torch.float16, "mfma_split": torch.float32}


def x16_prepare(values, indices, layout: Layout) -> torch.Tensor:
    """``nmg_x16_prepare``: the prepared operands of a packed weight (bytes)."""
    _need_cuda(values, indices)
    nbytes = lib().nmg_x16_prepared_bytes(layout.c)
    if nbytes < 0:
        raise NmgError(ERR_UNSUPPORTED, "nmg_x16_prepared_bytes")
    prepared = torch.empty(int(nbytes), dtype=torch.uint8, device=values.device)
    _check(lib().nmg_x16_prepare(layout.c, values.data_ptr(), indices.data_ptr(),
                                 prepared.data_ptr(), _stream(values)), "nmg_x16_prepare")
    return prepared


def spmm_x16_into(layout: Layout, prepared, X, Y):
    """``nmg_spmm_x16`` into a caller-allocated Y (M x N)."""
    _need_cuda(prepared, X, Y)
    if X.dtype != layout.dtype or Y.dtype != layout.dtype:
        raise TypeError("dtype mismatch")
    if X.shape[0] != layout.K or Y.shape[0] != layout.M or Y.shape[1] != X.shape[1]:
        raise ValueError("X must be K x N and Y M x N")
    _check(lib().nmg_spmm_x16(layout.c, prepared.data_ptr(), X.data_ptr(), _rows(X, "X"),
                              X.shape[1], Y.data_ptr(), _rows(Y, "Y"), _stream(X)), "nmg_spmm_x16")


def spmm_x16_epilogue(layout: Layout, prepared, X, epilogue: str = "none", R=None, Y=None):
    """``nmg_spmm_x16_epilogue``: Y = W_s X ("none") or W_s X + R ("add") from
    prepared operands, the sum taken as the product is stored."""
    _need_cuda(prepared, X)
    if X.dtype != layout.dtype or X.shape[0] != layout.K:
        raise ValueError("X must be K x N of the layout's dtype")
    N = X.shape[1]
    if Y is None:
        Y = X.new_empty((layout.M, N))
    _need_cuda(Y)
    if Y.dtype != layout.dtype or Y.shape != (layout.M, N):
        raise ValueError("Y must be M x N of the layout's dtype")
    rp, ldr = None, 0
    if epilogue == "add":
        if R is None:
            raise ValueError("the add epilogue needs R")
        _need_cuda(R)
        if R.dtype != layout.dtype or R.shape != (layout.M, N):
            raise ValueError("R must be M x N of the layout's dtype")
        rp, ldr = R.data_ptr(), _rows(R, "R")
    _check(lib().nmg_spmm_x16_epilogue(layout.c, prepared.data_ptr(),
                                       EPILOGUES[epilogue], X.data_ptr(), _rows(X, "X"), N, rp, ldr,
                                       Y.data_ptr(), _rows(Y, "Y"), _stream(X)),
           "nmg_spmm_x16_epilogue")
    return Y


def spmm_into(layout: Layout, values, indices, X, Y, kernel: str = "auto"):
    """``nmg_spmm_epilogue_ws`` without an epilogue into a caller-allocated Y
    (M x N), scratch memory from torch's allocator."""
    _need_cuda(values, indices, X, Y)
    if X.dtype != layout.dtype or Y.dtype != layout.dtype or values.dtype != layout.dtype:
        raise TypeError("dtype mismatch")
    if X.shape[0] != layout.K or Y.shape[0] != layout.M or Y.shape[1] != X.shape[1]:
        raise ValueError("X must be K x N and Y M x N")
    _packed_ok(layout, values, indices)
    L = lib()
    N, code = X.shape[1], KERNELS[kernel]
    vp, ip, xp, ldx = values.data_ptr(), indices.data_ptr(), X.data_ptr(), _rows(X, "X")
    ws, wp, wb = _workspace(_workspace_bytes(layout, code, vp, ip, xp, ldx, N), X)
    _check(L.nmg_spmm_epilogue_ws(layout.c, code, 0, vp, ip, xp, ldx, N, None, 0, Y.data_ptr(),
                                  _rows(Y, "Y"), wp, wb, _stream(X)), "nmg_spmm")


def spmm(values, indices, X, layout: Layout, kernel: str = "auto"):
    """Y = W_s X for the packed weight (values, indices)."""
    Y = X.new_empty((layout.M, X.shape[1]))
    spmm_into(layout, values, indices, X, Y, kernel)
    return Y


def spmm_epilogue(values, indices, X, layout: Layout, epilogue: str = "none", R=None,
                  kernel: str = "auto", Y=None):
    """Y = epilogue(W_s X): "none", "gelu" (GELU of the product) or "add"
    (product + R), bit for bit what spmm followed by gelu or add gives."""
    return _spmm_epilogue("nmg_spmm_epilogue_ws", values, indices, X, layout, epilogue, R, kernel, Y)


def spmm_epilogue_noalloc(values, indices, X, layout: Layout, epilogue: str = "none", R=None,
                          kernel: str = "auto", Y=None):
    """``nmg_spmm_epilogue_noalloc``: spmm_epilogue without device allocation
    in the library (the prepared operands of mfma_wide / mfma_split go to the
    library's fixed per-GPU array; overlapping calls on one GPU race).  "auto"
    never puts a layout into that array whose choice without a workspace has no
    scratch memory, so there spmm_epilogue, which brings a workspace, may take
    "sparse" where this call does not.  Y is
    allocated here when not given: pass Y to allocate nothing at all."""
    return _spmm_epilogue("nmg_spmm_epilogue_noalloc", values, indices, X, layout, epilogue, R,
                          kernel, Y)


def _spmm_epilogue(fn, values, indices, X, layout, epilogue, R, kernel, Y):
    _need_cuda(values, indices, X)
    if X.dtype != layout.dtype or values.dtype != layout.dtype:
        raise TypeError("dtype mismatch")
    if X.shape[0] != layout.K:
        raise ValueError("X must be K x N")
    _packed_ok(layout, values, indices)
    N = X.shape[1]
    if Y is None:
        Y = X.new_empty((layout.M, N))
    _need_cuda(Y)
    if Y.dtype != layout.dtype or Y.shape != (layout.M, N):
        raise ValueError("Y must be M x N of the layout's dtype")
    rp, ldr = None, 0
    if epilogue == "add":
        if R is None:
            raise ValueError("the add epilogue needs R")
        _need_cuda(R)
        if R.dtype != layout.dtype or R.shape != (layout.M, N):
            raise ValueError("R must be M x N of the layout's dtype")
        rp, ldr = R.data_ptr(), _rows(R, "R")
    L = lib()
    vp, ip, xp, ldx = values.data_ptr(), indices.data_ptr(), X.data_ptr(), _rows(X, "X")
    args = [layout.c, KERNELS[kernel], EPILOGUES[epilogue], vp, ip, xp, ldx, N, rp, ldr,
            Y.data_ptr(), _rows(Y, "Y")]
    if fn == "nmg_spmm_epilogue_ws":
        ws, wp, wb = _workspace(_workspace_bytes(layout, args[1], vp, ip, xp, ldx, N), X)
        args += [wp, wb]
    _check(getattr(L, fn)(*args, _stream(X)), fn)
    return Y


def auto_kernel(layout: Layout, N: int) -> str:
    """The family spmm / spmm_into / spmm_epilogue run for "auto" on aligned,
    contiguous operands (``nmg_spmm_plan``: they bring a workspace; the family
    without one is ``nmg_spmm_auto_kernel``)."""
    return _KERNEL_NAME[lib().nmg_spmm_plan(layout.c, KERNELS["auto"], None, None, None, N, N, None)]


def densify(values, indices, layout: Layout):
    """(values, indices) -> dense M x K weight (zeros at dropped positions)."""
    _need_cuda(values, indices)
    out = values.new_empty((layout.M, layout.K), dtype=layout.dtype)
    _check(lib().nmg_densify(layout.c, values.data_ptr(), indices.data_ptr(), out.data_ptr(),
                             layout.K, _stream(values)), "nmg_densify")
    return out


def gelu(x: torch.Tensor, out: torch.Tensor | None = None):
    _need_cuda(x)
    if not x.is_contiguous():
        raise ValueError("x must be contiguous")
    out = torch.empty_like(x) if out is None else out
    _check(lib().nmg_gelu(_DTYPE_CODE[x.dtype], x.data_ptr(), out.data_ptr(), x.numel(), _stream(x)),
           "nmg_gelu")
    return out


def add(a: torch.Tensor, b: torch.Tensor, out: torch.Tensor | None = None):
    _need_cuda(a, b)
    if a.shape != b.shape or a.dtype != b.dtype or not (a.is_contiguous() and b.is_contiguous()):
        raise ValueError("a and b must be contiguous tensors of one shape and dtype")
    out = torch.empty_like(a) if out is None else out
    _check(lib().nmg_add(_DTYPE_CODE[a.dtype], a.data_ptr(), b.data_ptr(), out.data_ptr(), a.numel(),
                         _stream(a)), "nmg_add")
    return out


# ------------------------------------------------ the paper's chunked layout

class PLayout:
    """Shape of one weight in the paper's chunked layout (``nmg_p_layout``)."""

    def __init__(self, M: int, K: int, n: int, m: int, g: int, dtype=torch.float32):
        if dtype not in _DTYPE_CODE:
            raise TypeError(f"unsupported dtype {dtype}")
        self.c = _PLayout()
        _check(lib().nmg_p_layout_init(ctypes.byref(self.c), M, K, n, m, g, _DTYPE_CODE[dtype]),
               "nmg_p_layout_init")
        self.dtype = dtype
        self._derive()

    def _derive(self):
        c = self.c
        self.M, self.K, self.n, self.m, self.g = c.M, c.K, c.n, c.m, c.g
        self.P, self.S, self.B = c.P, c.S, c.B
        self.values_shape = (self.M, self.B * self.n)
        self.index_shape = (self.M, self.B)

    def __setstate__(self, state):     # (also states of c and dtype alone)
        self.__dict__.update(state)
        self._derive()


def p_compress(W: torch.Tensor, n: int, m: int, g: int):
    """Dense W (M x K, GPU) -> (values, index, layout) in the chunked layout."""
    _need_cuda(W)
    layout = PLayout(W.shape[0], W.shape[1], n, m, g, W.dtype)
    values = W.new_empty(layout.values_shape)
    index = torch.empty(layout.index_shape, dtype=torch.uint8, device=W.device)
    _check(lib().nmg_p_compress(layout.c, W.data_ptr(), _rows(W, "W"), values.data_ptr(),
                                index.data_ptr(), _stream(W)), "nmg_p_compress")
    return values, index, layout


def _p_check(layout: PLayout, values, index):
    _need_cuda(values, index)
    if values.dtype != layout.dtype or index.dtype != torch.uint8:
        raise TypeError("dtype mismatch")
    if values.shape != layout.values_shape or not values.is_contiguous():
        raise ValueError(f"values must be contiguous {layout.values_shape}")
    if index.shape != layout.index_shape or not index.is_contiguous():
        raise ValueError(f"index must be contiguous {layout.index_shape}")


def p_spmm(values, index, X, layout: PLayout, kernel: str = "auto"):
    """Y = W_s X for the chunked layout; kernel is "auto", "valu" or "mfma"."""
    _p_check(layout, values, index)
    _need_cuda(X)
    if X.dtype != layout.dtype or X.shape[0] != layout.K:
        raise ValueError("X must be K x N of the layout's dtype")
    if kernel not in ("auto", "valu", "mfma"):
        raise ValueError(f"unknown chunked-layout kernel {kernel!r}")
    Y = X.new_empty((layout.M, X.shape[1]))
    L = lib()
    N, code = X.shape[1], KERNELS[kernel]
    ws, wp, wb = _workspace(L.nmg_p_spmm_workspace_bytes(layout.c, code, N), X)
    _check(L.nmg_p_spmm_ws(layout.c, code, values.data_ptr(), index.data_ptr(), X.data_ptr(),
                           _rows(X, "X"), N, Y.data_ptr(), _rows(Y, "Y"), wp, wb, _stream(X)),
           "nmg_p_spmm_ws")
    return Y


def p_densify(values, index, layout: PLayout):
    """Chunked layout -> dense M x K weight."""
    _p_check(layout, values, index)
    out = values.new_empty((layout.M, layout.K), dtype=layout.dtype)
    _check(lib().nmg_p_densify(layout.c, values.data_ptr(), index.data_ptr(), out.data_ptr(),
                               layout.K, _stream(values)), "nmg_p_densify")
    return out


def p_refine(W: torch.Tensor, index: torch.Tensor, layout: PLayout):
    """The swap search of Section 5.2's GPU converter from the packing `index`:
    returns new (values, index); the inputs are not changed."""
    _need_cuda(W, index)
    if W.dtype != layout.dtype or index.dtype != torch.uint8:
        raise TypeError("dtype mismatch")
    if W.shape != (layout.M, layout.K):
        raise ValueError(f"W must be {layout.M} x {layout.K}")
    if index.shape != layout.index_shape:
        raise ValueError(f"index must be {layout.index_shape}")
    idx = index.contiguous().clone()
    values = W.new_empty(layout.values_shape)
    _check(lib().nmg_p_refine(layout.c, W.data_ptr(), _rows(W, "W"), values.data_ptr(),
                              idx.data_ptr(), _stream(W)), "nmg_p_refine")
    return values, idx
