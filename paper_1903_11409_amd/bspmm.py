"""Thin binding of libbspmm.so: argument marshalling only, same names as the C ABI.

Plans and run calls go through ``_native.so`` (``csrc/binding.cpp``), everything else through ctypes.
Every step of the path (scheduling, staging, the products, the transposed build) runs inside
the library; PyTorch is used for device memory and streams only.  There is no fallback: if the
shared library is missing or a call fails, an exception is raised.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libbspmm.so")

OK, EINVAL, ENOSPACE, EHIP, EOVERLAP, ESTATE, EBADCSR, ETOOBIG = 0, -1, -2, -3, -4, -5, -6, -7
DRY_RUN, BUILD_TRANSPOSE, FLOOR_PROBE, SPLIT_HUB_ROWS, ACCUMULATE, COO_DIRECT, SYMMETRIC = 1, 2, 4, 8, 16, 32, 64
ONE_FRONT_LAUNCH = 128
BIN_WORKGROUP, BIN_WAVE, BIN_SLICE32, BIN_SLICE16, BIN_GENERIC = 0, 1, 2, 3, 4
NUM_BINS = 5
BIN_COO = 5          # items of a COO_DIRECT plan
BIN_NAMES = ["workgroup", "wave", "slice32", "slice16", "generic"]

_i32p = ctypes.POINTER(ctypes.c_int32)
_i64p = ctypes.POINTER(ctypes.c_int64)


class bspmm_batch(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int32),
                ("rows", _i32p), ("cols", _i32p), ("nnz", _i32p),
                ("rpt_off", _i64p), ("nz_off", _i64p), ("b_row_off", _i64p),
                ("c_row_off", _i64p),
                ("rpt", ctypes.c_void_p), ("colids", ctypes.c_void_p),
                ("values", ctypes.c_void_p)]


class bspmm_coo_batch(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int32),
                ("rows", _i32p), ("cols", _i32p), ("nnz", _i32p),
                ("nz_off", _i64p), ("b_row_off", _i64p), ("c_row_off", _i64p),
                ("ids", ctypes.c_void_p), ("values", ctypes.c_void_p)]


class bspmm_options(ctypes.Structure):
    _fields_ = [("flags", ctypes.c_uint32), ("force_bin", ctypes.c_int32),
                ("lds_bytes", ctypes.c_int32), ("min_tile", ctypes.c_int32),
                ("max_tile", ctypes.c_int32), ("target_workgroups", ctypes.c_int32),
                ("compute_units", ctypes.c_int32), ("lds_pad", ctypes.c_int32),
                ("max_passes", ctypes.c_int32), ("generic_rows", ctypes.c_int32),
                ("wg_passes", ctypes.c_int32), ("resident_workgroups", ctypes.c_int32),
                ("front_features", ctypes.c_int32), ("reserved_", ctypes.c_int32)]


class bspmm_info(ctypes.Structure):
    _fields_ = [("batch", ctypes.c_int32), ("F", ctypes.c_int32),
                ("lds_bytes", ctypes.c_int32), ("compute_units", ctypes.c_int32),
                ("tile", ctypes.c_int32 * 2), ("workgroups", ctypes.c_int32 * 2),
                ("tasks", ctypes.c_int32 * 2),
                ("items", ctypes.c_int32 * 2),
                ("items_in_bin", (ctypes.c_int32 * NUM_BINS) * 2),
                ("fused_tasks", ctypes.c_int32 * 2),
                ("transposed_supported", ctypes.c_int32),
                ("transposed_built", ctypes.c_int32),
                ("lean", ctypes.c_int32 * 2),
                ("front_stream", ctypes.c_int32 * 4),
                ("effective_bytes", ctypes.c_int64 * 2), ("flops", ctypes.c_int64),
                ("workspace_bytes", ctypes.c_uint64)]


class bspmm_kernel_resources(ctypes.Structure):
    _fields_ = [("vgprs", ctypes.c_int32), ("sgprs", ctypes.c_int32),
                ("static_lds_bytes", ctypes.c_int32), ("scratch_bytes", ctypes.c_int32),
                ("threads", ctypes.c_int32), ("workgroups_per_cu", ctypes.c_int32),
                ("compute_units", ctypes.c_int32), ("reserved_", ctypes.c_int32)]


class bspmm_item(ctypes.Structure):
    _fields_ = [("op", ctypes.c_int32), ("bin", ctypes.c_int32), ("row0", ctypes.c_int32),
                ("nrows", ctypes.c_int32), ("f0", ctypes.c_int32), ("fw", ctypes.c_int32),
                ("workgroup", ctypes.c_int32), ("slot", ctypes.c_int32)]


EXPORTS = ["bspmm_workspace_bytes", "bspmm_create", "bspmm_run", "bspmm_run_transposed",
           "bspmm_export_transposed", "bspmm_validate", "bspmm_plan_info", "bspmm_plan_items",
           "bspmm_destroy", "bspmm_strerror", "bspmm_last_hip_error",
           "bspmm_workspace_bytes_coo", "bspmm_create_coo", "bspmm_export_csr", "bspmm_run_gcn",
           "bspmm_create_static", "bspmm_kernel_info"]
KERNEL_NAMES = ["lean", "general", "general_scalar", "front", "layer", "build", "build_large", "coo",
                "layer_stream"]
STATIC_WORKSPACE_BYTES = 8 * 1024 * 1024

_lib = None
_native = None


class BspmmError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = int(code)
        msg = lib().bspmm_strerror(int(code)).decode()
        if code == EHIP:
            msg += f" (hipError {lib().bspmm_last_hip_error()})"
        super().__init__(f"{where}: {msg} [{code}]")


def lib():
    """The loaded shared library; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(
                f"{LIB_PATH} is missing: build it with `python -m paper_1903_11409_amd.build` "
                "(there is no fallback path)")
        L = ctypes.CDLL(LIB_PATH)
        vp = ctypes.c_void_p
        L.bspmm_workspace_bytes.argtypes = [ctypes.POINTER(bspmm_batch), ctypes.c_int32,
                                            ctypes.POINTER(bspmm_options),
                                            ctypes.POINTER(ctypes.c_size_t)]
        L.bspmm_create.argtypes = [ctypes.POINTER(vp), ctypes.POINTER(bspmm_batch),
                                   ctypes.c_int32, ctypes.POINTER(bspmm_options), vp,
                                   ctypes.c_size_t, vp]
        L.bspmm_create_static.argtypes = [ctypes.POINTER(vp), ctypes.POINTER(bspmm_batch),
                                          ctypes.c_int32, ctypes.POINTER(bspmm_options), vp]
        L.bspmm_run.argtypes = [vp, vp, vp, ctypes.c_int64, ctypes.c_int64, vp]
        L.bspmm_run_transposed.argtypes = [vp, vp, vp, ctypes.c_int64, ctypes.c_int64, vp]
        L.bspmm_export_transposed.argtypes = [vp, vp, vp, vp, vp]
        L.bspmm_validate.argtypes = [vp, _i32p, vp]
        L.bspmm_workspace_bytes_coo.argtypes = [ctypes.POINTER(bspmm_coo_batch), ctypes.c_int32,
                                                ctypes.POINTER(bspmm_options),
                                                ctypes.POINTER(ctypes.c_size_t)]
        L.bspmm_create_coo.argtypes = [ctypes.POINTER(vp), ctypes.POINTER(bspmm_coo_batch),
                                       ctypes.c_int32, ctypes.POINTER(bspmm_options), vp,
                                       ctypes.c_size_t, vp]
        L.bspmm_export_csr.argtypes = [vp, vp, vp, vp, vp]
        L.bspmm_run_gcn.argtypes = [vp, vp, ctypes.c_int64, vp, ctypes.c_int64, vp, vp,
                                    ctypes.c_int64, ctypes.c_int32, vp]
        L.bspmm_kernel_info.argtypes = [ctypes.c_int32, ctypes.c_int32,
                                        ctypes.POINTER(bspmm_kernel_resources)]
        L.bspmm_plan_info.argtypes = [vp, ctypes.POINTER(bspmm_info)]
        L.bspmm_plan_items.argtypes = [vp, ctypes.c_int32, ctypes.POINTER(bspmm_item),
                                       ctypes.c_int32, _i32p]
        L.bspmm_destroy.argtypes = [vp]
        L.bspmm_destroy.restype = None
        L.bspmm_strerror.argtypes = [ctypes.c_int]
        L.bspmm_strerror.restype = ctypes.c_char_p
        L.bspmm_last_hip_error.argtypes = []
        for n in EXPORTS:
            if n not in ("bspmm_destroy", "bspmm_strerror"):
                getattr(L, n).restype = ctypes.c_int
        _lib = L
    return _lib


def native():
    """The extension module of plans and run calls (``csrc/binding.cpp``); raises if it is not built."""
    global _native
    if _native is None:
        lib()
        import torch  # noqa: F401  (its libraries are what the module links against)
        try:
            from . import _native as module
        except ImportError as e:
            raise RuntimeError("_native.so is missing or does not load: build it with `python -m "
                               "paper_1903_11409_amd.build` (there is no fallback path)") from e
        module.setup(_check, _ld)
        _native = module
    return _native


def _check(code: int, where: str) -> None:
    if code != OK:
        raise BspmmError(code, where)


def _ptr(t) -> Optional[int]:
    """Device (or host) address of a torch tensor / raw integer; None stays NULL."""
    if t is None:
        return None
    if isinstance(t, int):
        return t
    return t.data_ptr()


def _ld(t, width: Optional[int]) -> int:
    """Leading dimension of a row-major matrix held in a tensor; a tensor with fewer than two
    rows (torch gives an empty one strides of zero) has none of its own and takes its width
    (``width`` None: nothing but its own)."""
    if width is None:
        width = t.shape[-1]
    if t.dim() != 2 or t.shape[0] < 2:
        return max(int(width), int(t.shape[-1]) if t.dim() else 0)
    return int(t.stride(0))


def _stream_handle(stream) -> Optional[int]:
    if stream is None:
        import torch
        return torch.cuda.current_stream().cuda_stream
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


def make_options(flags: int = 0, force_bin: Optional[int] = None, **kw) -> bspmm_options:
    """Options struct; ``force_bin`` takes a BIN_* constant (None = automatic)."""
    o = bspmm_options()
    o.flags = flags
    o.force_bin = 0 if force_bin is None else 1 + int(force_bin)
    for k, v in kw.items():
        if not hasattr(o, k):
            raise TypeError(f"unknown option {k}")
        setattr(o, k, int(v))
    return o


class HostBatch:
    """Keeps the numpy metadata arrays alive and exposes them as a ``bspmm_batch``."""

    def __init__(self, rows, cols, nnz, rpt_off, nz_off, b_row_off, c_row_off,
                 rpt_dev=None, colids_dev=None, values_dev=None):
        as_ = np.ascontiguousarray
        self.arrays = [as_(rows, dtype=np.int32), as_(cols, dtype=np.int32),
                       as_(nnz, dtype=np.int32), as_(rpt_off, dtype=np.int64),
                       as_(nz_off, dtype=np.int64), as_(b_row_off, dtype=np.int64),
                       as_(c_row_off, dtype=np.int64)]
        self.device = (rpt_dev, colids_dev, values_dev)
        s = bspmm_batch()
        s.batch = int(self.arrays[0].shape[0])
        a = self.arrays
        s.rows = a[0].ctypes.data_as(_i32p)
        s.cols = a[1].ctypes.data_as(_i32p)
        s.nnz = a[2].ctypes.data_as(_i32p)
        s.rpt_off = a[3].ctypes.data_as(_i64p)
        s.nz_off = a[4].ctypes.data_as(_i64p)
        s.b_row_off = a[5].ctypes.data_as(_i64p)
        s.c_row_off = a[6].ctypes.data_as(_i64p)
        s.rpt = _ptr(rpt_dev)
        s.colids = _ptr(colids_dev)
        s.values = _ptr(values_dev)
        self.struct = s


class HostCooBatch:
    """Keeps the numpy metadata arrays alive and exposes them as a ``bspmm_coo_batch``."""

    def __init__(self, rows, cols, nnz, nz_off, b_row_off, c_row_off, ids_dev=None,
                 values_dev=None):
        as_ = np.ascontiguousarray
        self.arrays = [as_(rows, dtype=np.int32), as_(cols, dtype=np.int32),
                       as_(nnz, dtype=np.int32), as_(nz_off, dtype=np.int64),
                       as_(b_row_off, dtype=np.int64), as_(c_row_off, dtype=np.int64)]
        self.device = (ids_dev, values_dev)
        s = bspmm_coo_batch()
        a = self.arrays
        s.batch = int(a[0].shape[0])
        s.rows = a[0].ctypes.data_as(_i32p)
        s.cols = a[1].ctypes.data_as(_i32p)
        s.nnz = a[2].ctypes.data_as(_i32p)
        s.nz_off = a[3].ctypes.data_as(_i64p)
        s.b_row_off = a[4].ctypes.data_as(_i64p)
        s.c_row_off = a[5].ctypes.data_as(_i64p)
        s.ids = _ptr(ids_dev)
        s.values = _ptr(values_dev)
        self.struct = s


def bspmm_workspace_bytes_coo(hb: HostCooBatch, F: int,
                              options: Optional[bspmm_options] = None) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().bspmm_workspace_bytes_coo(ctypes.byref(hb.struct), int(F),
                                           ctypes.byref(options) if options is not None else None,
                                           ctypes.byref(out)), "bspmm_workspace_bytes_coo")
    return int(out.value)


def bspmm_create_coo(hb: HostCooBatch, F: int, options: Optional[bspmm_options] = None,
                     workspace=None, workspace_bytes: int = 0, stream=None) -> int:
    """Returns the opaque plan handle (an integer address)."""
    plan = ctypes.c_void_p(None)
    dry = options is not None and (options.flags & DRY_RUN)
    _check(lib().bspmm_create_coo(ctypes.byref(plan), ctypes.byref(hb.struct), int(F),
                                  ctypes.byref(options) if options is not None else None,
                                  _ptr(workspace), int(workspace_bytes),
                                  None if dry else _stream_handle(stream)), "bspmm_create_coo")
    return plan.value


def bspmm_export_csr(plan: int, rpt, colids, values, stream=None) -> None:
    _check(lib().bspmm_export_csr(plan, _ptr(rpt), _ptr(colids), _ptr(values),
                                  _stream_handle(stream)), "bspmm_export_csr")


def bspmm_workspace_bytes(hb: HostBatch, F: int, options: Optional[bspmm_options] = None) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().bspmm_workspace_bytes(ctypes.byref(hb.struct), int(F),
                                       ctypes.byref(options) if options is not None else None,
                                       ctypes.byref(out)), "bspmm_workspace_bytes")
    return int(out.value)


def bspmm_create(hb: HostBatch, F: int, options: Optional[bspmm_options] = None,
                 workspace=None, workspace_bytes: int = 0, stream=None) -> int:
    """Returns the opaque plan handle (an integer address)."""
    plan = ctypes.c_void_p(None)
    dry = options is not None and (options.flags & DRY_RUN)
    _check(lib().bspmm_create(ctypes.byref(plan), ctypes.byref(hb.struct), int(F),
                              ctypes.byref(options) if options is not None else None,
                              _ptr(workspace), int(workspace_bytes),
                              None if dry else _stream_handle(stream)), "bspmm_create")
    return plan.value


def bspmm_create_static(hb: HostBatch, F: int, options: Optional[bspmm_options] = None,
                        stream=None) -> int:
    """Plan whose workspace is the library's static device array; returns the plan handle."""
    plan = ctypes.c_void_p(None)
    _check(lib().bspmm_create_static(ctypes.byref(plan), ctypes.byref(hb.struct), int(F),
                                     ctypes.byref(options) if options is not None else None,
                                     _stream_handle(stream)), "bspmm_create_static")
    return plan.value


def bspmm_run(plan: int, B, C, ldb: int, ldc: int, stream=None) -> None:
    (_native or native()).run(plan, B, C, int(ldb), int(ldc), stream)


def bspmm_run_gcn(plan: int, X, ldx: int, W, ldw: int, bias, Y, ldy: int, accumulate: bool = False,
                  stream=None) -> None:
    (_native or native()).run_gcn(plan, X, W, bias, Y, int(ldx), int(ldw), int(ldy), accumulate, stream)


def bspmm_run_transposed(plan: int, dY, G, ldy: int, ldg: int, stream=None) -> None:
    (_native or native()).run_transposed(plan, dY, G, int(ldy), int(ldg), stream)


def bspmm_export_transposed(plan: int, rpt_t, colids_t, values_t, stream=None) -> None:
    _check(lib().bspmm_export_transposed(plan, _ptr(rpt_t), _ptr(colids_t), _ptr(values_t),
                                         _stream_handle(stream)), "bspmm_export_transposed")


def bspmm_validate(plan: int, stream=None) -> int:
    """Returns -1 when the device CSR is well formed, else the first malformed operation."""
    bad = ctypes.c_int32(-1)
    rc = lib().bspmm_validate(plan, ctypes.byref(bad), _stream_handle(stream))
    if rc == EBADCSR:
        return int(bad.value)
    _check(rc, "bspmm_validate")
    return -1


def bspmm_kernel_info(kernel: int, dynamic_lds_bytes: int = 0) -> bspmm_kernel_resources:
    out = bspmm_kernel_resources()
    _check(lib().bspmm_kernel_info(int(kernel), int(dynamic_lds_bytes), ctypes.byref(out)),
           "bspmm_kernel_info")
    return out


def bspmm_plan_info(plan: int) -> bspmm_info:
    info = bspmm_info()
    _check(lib().bspmm_plan_info(plan, ctypes.byref(info)), "bspmm_plan_info")
    return info


def bspmm_plan_items(plan: int, transposed: bool = False):
    n = ctypes.c_int32(0)
    _check(lib().bspmm_plan_items(plan, int(bool(transposed)), None, 0, ctypes.byref(n)),
           "bspmm_plan_items")
    arr = (bspmm_item * max(n.value, 1))()
    _check(lib().bspmm_plan_items(plan, int(bool(transposed)), arr, n.value, ctypes.byref(n)),
           "bspmm_plan_items")
    return [arr[i] for i in range(n.value)]


def bspmm_destroy(plan: Optional[int]) -> None:
    if plan:
        lib().bspmm_destroy(plan)


class Plan:
    """Owns a plan handle plus the torch tensors it borrows (CSR arrays and workspace).

    ``batch`` is a :class:`workloads.Batch`-like object: the per-operation sizes and offsets are
    host arrays; the CSR arrays (``rpt``, ``colids``, ``values``) are numpy arrays, copied to
    ``device`` once, or tensors already there, borrowed in place.  Dense operands are passed per
    call as torch tensors.
    """

    def __init__(self, batch, F: Optional[int] = None, options: Optional[bspmm_options] = None,
                 device="cuda:0", stream=None, coo=None):
        import torch
        n = _native or native()
        self.torch = torch
        self.n_x = max(1, int(options.front_features)) if options is not None else 1
        self.F = int(F if F is not None else batch.F)
        self._hb = self._views = None
        self.device = device = torch.device(device)
        index = device.index if device.index is not None else torch.cuda.current_device()
        self.options = options
        opt = None if options is None else ctypes.addressof(options)
        self._meta = meta = (batch.rows, batch.cols, batch.nnz, getattr(batch, "rpt_off", None), batch.nz_off,
                             batch.b_row_off, batch.c_row_off)
        if coo is not None:
            # COO / SparseTensor operands: ``coo`` = (ids, values), numpy arrays or tensors, laid
            # out by the batch's nz_off; the batch's own CSR arrays are not used
            ids, values = coo
            self._csr = None
            made = n.create_coo(*meta[:3], *meta[4:], ids, values, self.F, opt, index, stream)
            if made is None:
                self._meta = meta = self._as_arrays(meta[:3], np.int32) + (None,) + self._as_arrays(meta[4:], np.int64)
                ids, values = self._on_device(ids, torch.int32), self._on_device(values, torch.float32)
                made = n.create_coo(*meta[:3], *meta[4:], ids, values, self.F, opt, index, stream)
            self.ids, self.values = ids, values
        else:
            csr = (batch.rpt, batch.colids, batch.values)
            made = n.create(*meta, *csr, self.F, opt, index, stream)
            if made is None:      # another type or layout, on another device, or too large to be staged
                self._meta = meta = self._as_arrays(meta[:3], np.int32) + self._as_arrays(meta[3:], np.int64)
                rpt, colids, values = (self._on_device(a, t) for a, t in zip(csr, (torch.int32, torch.int32,
                                                                                    torch.float32)))
                # zero-length tensors have a null data_ptr; give the library something addressable
                if rpt.numel() == 0:
                    rpt = torch.zeros(1, dtype=torch.int32, device=device)
                csr = (rpt, colids, values)
                made = n.create(*meta, *csr, self.F, opt, index, stream)
            self._csr = csr       # as given, or as lengths of the arrays in front of the workspace
            if made is not None and made[2] > 0:
                self._csr = tuple(int(a.shape[0]) for a in csr)
        if made is None:
            raise TypeError("the batch's arrays cannot be used: one-dimensional arrays of one length are needed")
        self.handle, self._memory, self._head, self.rpt_len, self.rpt_t_len, self.nnz_total = made

    @staticmethod
    def _as_arrays(arrays, dtype):
        return tuple(np.ascontiguousarray(a, dtype=dtype).reshape(-1) for a in arrays)

    def _on_device(self, a, dtype):
        # numpy arrays are copied over; tensors that already sit on the device with the
        # right type and layout are borrowed as they are
        torch = self.torch
        if isinstance(a, torch.Tensor):
            return a.to(device=self.device, dtype=dtype).contiguous()
        np_type = np.int32 if dtype == torch.int32 else np.float32
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np_type)).to(self.device)

    def __getattr__(self, name):
        # what only inspection asks for is made when it is asked for
        if name == "hb":
            if self._hb is None:
                m = self._meta
                if self._csr is None:
                    self._hb = HostCooBatch(*m[:3], *m[4:], self.ids if self.ids.numel() else None,
                                            self.values if self.values.numel() else None)
                else:
                    self._hb = HostBatch(*m, self.rpt, self.colids if self.colids.numel() else None,
                                         self.values if self.values.numel() else None)
            return self._hb
        if name == "workspace":
            return self._memory[self._head:]
        if name in ("rpt", "colids", "values") and self.__dict__.get("_csr") is not None:
            if self._views is None:
                self._views = self._csr
                if self._head > 0:
                    at, views = 0, []
                    for n, t in zip(self._csr, (self.torch.int32, self.torch.int32, self.torch.float32)):
                        views.append(self._memory[at:at + 4 * n].view(t))
                        at += (4 * n + 255) // 256 * 256
                    self._views = tuple(views)
            return self._views[("rpt", "colids", "values").index(name)]
        raise AttributeError(name)

    def run(self, B, C, stream=None):
        return _native.plan_run(self.handle, B, C, self.F, stream)

    def run_gcn(self, X, W, bias, Y, accumulate: bool = False, stream=None):
        """Y (+)= A (X W + bias) in one launch (plan created with ``front_features``)."""
        return _native.plan_run_gcn(self.handle, X, W, bias, Y, self.n_x, self.F, accumulate, stream)

    def run_transposed(self, dY, G, stream=None):
        return _native.plan_run_transposed(self.handle, dY, G, self.F, stream)

    def covered_rows(self, transposed: bool = False) -> int:
        """Rows from the first on that every product writes: C's, or G's when ``transposed``."""
        return _native.covered_rows(self.handle, transposed)

    def export_transposed(self, stream=None):
        t = self.torch
        rpt_t = t.empty(max(self.rpt_t_len, 1), dtype=t.int32, device=self.device)
        col_t = t.empty(max(self.nnz_total, 1), dtype=t.int32, device=self.device)
        val_t = t.empty(max(self.nnz_total, 1), dtype=t.float32, device=self.device)
        bspmm_export_transposed(self.handle, rpt_t, col_t, val_t, stream)
        return rpt_t[:self.rpt_t_len], col_t[:self.nnz_total], val_t[:self.nnz_total]

    def export_csr(self, stream=None):
        """CSR arrays a COO plan built on the device (rpt, colids, values)."""
        t = self.torch
        rpt = t.empty(max(self.rpt_len, 1), dtype=t.int32, device=self.device)
        col = t.empty(max(self.nnz_total, 1), dtype=t.int32, device=self.device)
        val = t.empty(max(self.nnz_total, 1), dtype=t.float32, device=self.device)
        bspmm_export_csr(self.handle, rpt, col, val, stream)
        return rpt[:self.rpt_len], col[:self.nnz_total], val[:self.nnz_total]

    def validate(self, stream=None) -> int:
        return bspmm_validate(self.handle, stream)

    def info(self) -> bspmm_info:
        return bspmm_plan_info(self.handle)

    def items(self, transposed: bool = False):
        return bspmm_plan_items(self.handle, transposed)

    def close(self):
        if getattr(self, "handle", None):
            bspmm_destroy(self.handle)
            self.handle = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def dry_plan(batch, F: Optional[int] = None, **option_kw) -> int:
    """Schedule-only plan (no device needed); free it with bspmm_destroy."""
    kw = dict(option_kw)
    flags = kw.pop("flags", 0) | DRY_RUN
    coo = kw.pop("coo", False)
    opts = make_options(flags=flags, **kw)
    if coo:
        hc = HostCooBatch(batch.rows, batch.cols, batch.nnz, batch.nz_off, batch.b_row_off,
                          batch.c_row_off)
        return bspmm_create_coo(hc, int(F if F is not None else batch.F), opts)
    hb = HostBatch(batch.rows, batch.cols, batch.nnz, batch.rpt_off, batch.nz_off,
                   batch.b_row_off, batch.c_row_off)
    return bspmm_create(hb, int(F if F is not None else batch.F), opts)
