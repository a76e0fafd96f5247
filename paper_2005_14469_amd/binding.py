"""Binding of include/gcoo.h: argument marshalling only, by ctypes, and for the calls of every matrix and product by the
extension module _calls (csrc_python/calls.cpp) where that is built and the arguments are as it expects them.

Every step of the path (conversion to GCOO and the product) runs in the HIP kernels of
libgcoo.so.  torch is used for device memory and for the current stream, nothing else.  If
the library has not been built, loading it raises: there is no fallback.
"""
from __future__ import annotations

import contextlib
import ctypes as C
import os
import warnings

import numpy as np
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# GCOO_LIBRARY names another build of the same library (the host-sanitized one of build.py --host-sanitize)
LIB_PATH = os.environ.get("GCOO_LIBRARY") or os.path.join(_HERE, "libgcoo.so")
CALLS_PATH = os.path.join(_HERE, "_calls.so")
BASELINE_LIB_PATH = os.path.join(_HERE, "libgcoo_baseline.so")

GCOO_OK, GCOO_EINVAL, GCOO_EBOUNDS, GCOO_ENOMEM, GCOO_EHIP, GCOO_ELIMIT = 0, -1, -2, -3, -4, -5
GCOO_STATIC_MAX_NNZ = 2097152
GCOO_MAX_P = 256
VARIANT_AUTO, VARIANT_LDS, VARIANT_REG, VARIANT_SHARE = 0, 1, 2, 3
KERNEL_NONE, KERNEL_LDS, KERNEL_SCHED, KERNEL_SHARE, KERNEL_ROWS, KERNEL_BAND = 0, 1, 2, 3, 4, 5
SHARE_AUTO, SHARE_ALWAYS, SHARE_NEVER = 0, 1, 2

# every symbol include/gcoo.h declares
SYMBOLS = ["gcoo_default_p", "gcoo_device_bytes", "gcoo_from_csr", "gcoo_from_csr_device", "gcoo_dense_nnz", "gcoo_from_dense", "gcoo_spdm",
           "gcoo_dense_count_bytes", "gcoo_dense_count", "gcoo_from_dense_counted",
           "gcoo_spdm_variant", "gcoo_spdm_pick", "gcoo_spdm_kernel", "gcoo_free", "gcoo_info", "gcoo_export",
           "gcoo_strerror", "gcoo_last_hip_error", "gcoo_set_share_policy", "gcoo_export_share",
           "gcoo_static_handle_bytes", "gcoo_from_csr_device_static"]
# and include/gcoo_baseline.h (libgcoo_baseline.so)
BASELINE_SYMBOLS = ["gcoo_csr_spmm_baseline"]

_lib = None
_calls = None              # the extension module, or what stands for it: there as soon as lib() has been called
_baseline_lib = None


class GcooError(RuntimeError):
    def __init__(self, status: int, where: str):
        L = lib()
        msg = L.gcoo_strerror(status).decode()
        if status == GCOO_EHIP:
            msg += ": " + L.gcoo_last_hip_error().decode()
        super().__init__(f"{where}: {msg} ({status})")
        self.status = status


class _ByCtypes:
    """In the place of an extension module that is not there: serves no call, so that all of them go by ctypes."""

    @staticmethod
    def free(handle):
        lib().gcoo_free(handle)

    from_csr_device = from_csr_host = from_csr_device_static = from_dense = spdm = staticmethod(lambda *args: None)


def lib():
    """Load libgcoo.so (built in-tree by paper_2005_14469_amd/build.py)."""
    global _lib, _calls
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(
                f"{LIB_PATH} is missing: build it with `python -m paper_2005_14469_amd.build` "
                "(there is no CPU fallback)")
        calls = _ByCtypes
        # (in front of the library: with the two the other way round in memory every call took the host 0.5 us more in most processes; 256 x 256, 10 %, N = 256, a step: 9.6 and 10.7 us)
        if os.path.exists(CALLS_PATH):
            from . import _calls as calls
        L = C.CDLL(LIB_PATH)
        i64, i32, vp, sz = C.c_int64, C.c_int32, C.c_void_p, C.c_size_t
        L.gcoo_device_bytes.restype = sz
        L.gcoo_device_bytes.argtypes = [i64, i64, i64, i32]
        L.gcoo_from_csr.restype = C.c_int
        L.gcoo_from_csr.argtypes = [i64, i64, vp, vp, vp, C.c_int, i32, vp, sz, vp, C.POINTER(vp)]
        L.gcoo_dense_nnz.restype = C.c_int
        L.gcoo_dense_nnz.argtypes = [i64, i64, vp, i64, vp, C.POINTER(i64)]
        L.gcoo_from_dense.restype = C.c_int
        L.gcoo_from_dense.argtypes = [i64, i64, vp, i64, i32, vp, sz, vp, C.POINTER(vp)]
        L.gcoo_dense_count_bytes.restype = sz
        L.gcoo_dense_count_bytes.argtypes = [i64, i64, i32]
        L.gcoo_dense_count.restype = C.c_int
        L.gcoo_dense_count.argtypes = [i64, i64, vp, i64, i32, vp, sz, vp, C.POINTER(i64)]
        L.gcoo_from_dense_counted.restype = C.c_int
        L.gcoo_from_dense_counted.argtypes = [i64, i64, i64, vp, i64, i32, vp, vp, sz, vp, C.POINTER(vp)]
        L.gcoo_spdm.restype = C.c_int
        L.gcoo_spdm.argtypes = [vp, vp, i64, i64, vp, i64, vp]
        L.gcoo_spdm_variant.restype = C.c_int
        L.gcoo_spdm_variant.argtypes = [vp, vp, i64, i64, vp, i64, vp, C.c_int]
        L.gcoo_spdm_pick.restype = C.c_int
        L.gcoo_spdm_pick.argtypes = [vp, vp, i64, i64, vp, i64]
        L.gcoo_spdm_kernel.restype = C.c_int
        L.gcoo_spdm_kernel.argtypes = [vp, vp, i64, i64, vp, i64, C.c_int]
        L.gcoo_free.restype = C.c_int
        L.gcoo_free.argtypes = [vp]
        L.gcoo_info.restype = C.c_int
        L.gcoo_info.argtypes = [vp, C.POINTER(i64), C.POINTER(i64), C.POINTER(i64), C.POINTER(i32), C.POINTER(i64)]
        L.gcoo_export.restype = C.c_int
        L.gcoo_export.argtypes = [vp, vp, vp, vp, vp, vp, vp]
        L.gcoo_from_csr_device.restype = C.c_int
        L.gcoo_from_csr_device.argtypes = [i64, i64, i64, vp, vp, vp, i32, vp, C.c_size_t, vp, C.POINTER(vp)]
        L.gcoo_static_handle_bytes.restype = sz
        L.gcoo_static_handle_bytes.argtypes = [i64, i64, i64, i32]
        L.gcoo_from_csr_device_static.restype = C.c_int
        L.gcoo_from_csr_device_static.argtypes = [i64, i64, i64, vp, vp, vp, i32, vp, C.c_size_t, vp, C.POINTER(vp)]
        L.gcoo_set_share_policy.restype = C.c_int
        L.gcoo_set_share_policy.argtypes = [C.c_int]
        L.gcoo_export_share.restype = C.c_int
        L.gcoo_export_share.argtypes = [vp, vp, vp, vp, vp, vp, C.POINTER(i64), C.POINTER(i64), vp]
        L.gcoo_default_p.restype = C.c_int32
        L.gcoo_default_p.argtypes = [i64, i64, i64, i64]
        L.gcoo_strerror.restype = C.c_char_p
        L.gcoo_strerror.argtypes = [C.c_int]
        L.gcoo_last_hip_error.restype = C.c_char_p
        L.gcoo_last_hip_error.argtypes = []
        if calls is not _ByCtypes:
            calls.bind(*(C.cast(getattr(L, name), vp).value for name in
                          ("gcoo_device_bytes", "gcoo_from_csr", "gcoo_from_csr_device", "gcoo_from_csr_device_static", "gcoo_dense_count_bytes", "gcoo_dense_count",
                           "gcoo_from_dense_counted", "gcoo_spdm_variant", "gcoo_free")))
        _calls = calls
        _lib = L
        if calls is _ByCtypes:
            warnings.warn(f"{CALLS_PATH} is missing: all calls go by ctypes, with the same results (`python -m paper_2005_14469_amd.build` builds it)", RuntimeWarning, stacklevel=2)
    return _lib


def baseline_lib():
    """Load libgcoo_baseline.so (the CSR row-split routine the benchmark compares against)."""
    global _baseline_lib
    if _baseline_lib is None:
        if not os.path.exists(BASELINE_LIB_PATH):
            raise FileNotFoundError(f"{BASELINE_LIB_PATH} is missing: build it with `python -m paper_2005_14469_amd.build`")
        L = C.CDLL(BASELINE_LIB_PATH)
        i64, vp = C.c_int64, C.c_void_p
        L.gcoo_csr_spmm_baseline.restype = C.c_int
        L.gcoo_csr_spmm_baseline.argtypes = [i64, i64, vp, vp, vp, vp, i64, i64, vp, i64, vp]
        _baseline_lib = L
    return _baseline_lib


def _check(status: int, where: str):
    if status != GCOO_OK:
        raise GcooError(status, where)


# A product of a small matrix takes the device less time than Python needs for a torch.cuda.Stream object, a device context and
# an info() (2.6, 1.2 and 1.2 us; the whole of gcoo_spdm() took 10.2 us for 400 x 400, of which 3.9 in the library): the calls below ask
# for the raw stream, switch devices only where the tensors are elsewhere, and keep a matrix's shape with its handle.  What they do first is to leave a call of ordinary arguments on the
# current stream to the extension module, which returns None for any other, a status, or the result.
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None) or (lambda d: torch.cuda.current_stream(d).cuda_stream)
_no_switch = contextlib.nullcontext()


def _stream_ptr(stream=None):
    return stream.cuda_stream if stream is not None else _raw_stream(torch.cuda.current_device())


def _on(device_index: int):
    """The context in which `device_index` is current."""
    return _no_switch if device_index == torch.cuda.current_device() else torch.cuda.device(device_index)


def _used_on(t: torch.Tensor, stream) -> None:
    """`t`, of the current stream's memory, is used by kernels on `stream`: once it is dropped its memory is given out again only behind them.  (That `stream`
    is ordered behind what the current one has done so far is the caller's part, as everywhere in torch.)"""
    t.record_stream(stream if isinstance(stream, torch.Stream) else torch.cuda.ExternalStream(stream.cuda_stream, device=t.device))


def gcoo_device_bytes(m: int, k: int, nnz: int, p: int) -> int:
    return int(lib().gcoo_device_bytes(m, k, nnz, p))


class GcooMatrix:
    """Owner of one handle and of the torch buffer behind it."""

    def __init__(self, handle, buf: torch.Tensor):
        self._h = handle.value if isinstance(handle, C.c_void_p) else handle          # the address: what the extension module takes
        self.buf = buf
        self._mk = None

    @property
    def shape(self):
        if self._mk is None:
            i = self.info()
            self._mk = (i["m"], i["k"])
        return self._mk

    def _address(self) -> int:
        if self._h is None:
            raise ValueError("handle already freed")
        return self._h

    @property
    def handle(self) -> C.c_void_p:
        """For a call of the C ABI: a pointer also for a function of which ctypes has not been told the types."""
        return C.c_void_p(self._address())

    def info(self):
        m, k, nnz, g = C.c_int64(), C.c_int64(), C.c_int64(), C.c_int64()
        p = C.c_int32()
        _check(lib().gcoo_info(self.handle, C.byref(m), C.byref(k), C.byref(nnz), C.byref(p), C.byref(g)), "gcoo_info")
        return dict(m=m.value, k=k.value, nnz=nnz.value, p=p.value, g=g.value)

    def export(self, stream=None):
        """The five arrays as numpy arrays on the host (gIdxes has g+1 int64 entries)."""
        i = self.info()
        v = np.empty(i["nnz"], np.float32)
        r = np.empty(i["nnz"], np.int32)
        c = np.empty(i["nnz"], np.int32)
        gi = np.empty(i["g"] + 1, np.int64)
        npg = np.empty(i["g"], np.int32)
        _check(lib().gcoo_export(self.handle, v.ctypes.data, r.ctypes.data, c.ctypes.data, gi.ctypes.data,
                                 npg.ctypes.data, _stream_ptr(stream)), "gcoo_export")
        return dict(values=v, rows=r, cols=c, gIdxes=gi, nnzPerGroup=npg)

    def export_share(self, stream=None):
        """The share schedule as numpy arrays on the host; arrays of no elements where VARIANT_SHARE reads the band schedule instead;
        None for a matrix that VARIANT_SHARE does not serve."""
        hw, nb = C.c_int64(), C.c_int64()
        if lib().gcoo_export_share(self.handle, None, None, None, None, None, C.byref(hw), C.byref(nb), _stream_ptr(stream)) != GCOO_OK:
            return None
        if hw.value == 0:
            return dict(hdr=np.empty(0, np.uint32), blocks=np.empty(0, np.uint32), sbase=np.empty(0, np.int32), ucount=np.empty(0, np.int32),
                        ucols=np.empty(0, np.int32))
        i = self.info()
        nq = (i["g"] + 7) // 8
        hdr = np.empty(hw.value, np.uint32)
        blocks = np.empty(nb.value * 64, np.uint32)
        sbase = np.empty(nq * 8, np.int32)
        ucount = np.empty(nq, np.int32)
        ucols = np.empty(i["nnz"], np.int32)
        _check(lib().gcoo_export_share(self.handle, hdr.ctypes.data, blocks.ctypes.data, sbase.ctypes.data, ucount.ctypes.data,
                                       ucols.ctypes.data, None, None, _stream_ptr(stream)), "gcoo_export_share")
        return dict(hdr=hdr, blocks=blocks, sbase=sbase, ucount=ucount, ucols=ucols)

    def free(self):
        if self._h is not None:
            _calls.free(self._h) if _calls else lib().gcoo_free(self._h)
            self._h = None
            self.buf = None

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


def _module():
    lib()
    return _calls


def _matrix(got, shape, where: str) -> GcooMatrix:
    """What a conversion of the extension module returned: a handle and its buffer, or a status."""
    if type(got) is int:
        raise GcooError(got, where)
    A = GcooMatrix(*got)
    A._mk = shape
    return A


def _alloc(nbytes: int, device) -> torch.Tensor:
    buf = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=device)
    assert buf.data_ptr() % 256 == 0
    return buf


def gcoo_from_csr(m: int, k: int, row_ptr, col_idx, vals, p: int, device="cuda:0", stream=None,
                  known_nnz: bool = False) -> GcooMatrix:
    """row_ptr/col_idx/vals: numpy arrays (host input) or torch device tensors (device input).

    known_nnz (device input only): the caller vouches that row_ptr[m] == len(col_idx); the
    conversion then reads nothing back and never waits for the device (gcoo_from_csr_device)."""
    on_dev = isinstance(row_ptr, torch.Tensor)
    if not on_dev:
        device = torch.device(device)
        assert device.type == "cuda"
    if stream is None:
        calls, got = _calls or _module(), None
        if on_dev:
            if row_ptr.is_cuda:
                got = calls.from_csr_device(row_ptr, col_idx, vals, m, k, p, _raw_stream(row_ptr.get_device()), known_nnz)
        else:
            current = torch.cuda.current_device()
            if device.index is None or device.index == current:
                got = calls.from_csr_host(row_ptr, col_idx, vals, m, k, p, _raw_stream(current))
        if got is not None:
            return _matrix(got, (m, k), "gcoo_from_csr_device" if on_dev and known_nnz else "gcoo_from_csr")
    if on_dev:
        assert row_ptr.is_cuda and row_ptr.dtype == torch.int32 and row_ptr.is_contiguous()
        assert col_idx.dtype == torch.int32 and vals.dtype == torch.float32
        nnz = col_idx.numel()
        ptrs = (row_ptr.data_ptr(), col_idx.data_ptr(), vals.data_ptr())
        device, index = row_ptr.device, row_ptr.get_device()
    else:
        row_ptr = np.ascontiguousarray(row_ptr, dtype=np.int32)
        col_idx = np.ascontiguousarray(col_idx, dtype=np.int32)
        vals = np.ascontiguousarray(vals, dtype=np.float32)
        nnz = int(col_idx.shape[0])
        ptrs = (row_ptr.ctypes.data, col_idx.ctypes.data, vals.ctypes.data)
        index = torch.cuda.current_device() if device.index is None else device.index
    L = lib()
    need = L.gcoo_device_bytes(m, k, nnz, p)
    if need == 0:
        raise GcooError(GCOO_EINVAL, "gcoo_device_bytes")
    with _on(index):
        buf = _alloc(need, device)
        if stream is not None:
            _used_on(buf, stream)
        out = C.c_void_p()
        sp = _raw_stream(index) if stream is None else stream.cuda_stream
        if on_dev and known_nnz:
            status = L.gcoo_from_csr_device(m, k, nnz, *ptrs, p, buf.data_ptr(), need, sp, C.byref(out))
        else:
            status = L.gcoo_from_csr(m, k, *ptrs, 1 if on_dev else 0, p, buf.data_ptr(), need, sp, C.byref(out))
    if status:
        raise GcooError(status, "gcoo_from_csr_device" if on_dev and known_nnz else "gcoo_from_csr")
    A = GcooMatrix(out, buf)
    A._mk = (m, k)
    return A


def gcoo_from_csr_device_static(m: int, k: int, row_ptr: torch.Tensor, col_idx: torch.Tensor, vals: torch.Tensor, p: int,
                                out_buf: torch.Tensor | None = None, stream=None) -> GcooMatrix:
    """gcoo_from_csr_device_static: the conversion that allocates no device memory.  out_buf (a uint8 device
    tensor the caller already owns) receives what the handle keeps; without one, a tensor of
    gcoo_static_handle_bytes is made here first (the C call itself allocates nothing either way)."""
    if stream is None and out_buf is not None and row_ptr.is_cuda:
        got = (_calls or _module()).from_csr_device_static(row_ptr, col_idx, vals, m, k, p, out_buf, _raw_stream(row_ptr.get_device()))
        if got is not None:
            return _matrix((got, out_buf) if type(got) is int else got[0], (m, k), "gcoo_from_csr_device_static")
    assert row_ptr.is_cuda and row_ptr.dtype == torch.int32 and col_idx.dtype == torch.int32 and vals.dtype == torch.float32
    nnz = int(col_idx.numel())
    need = int(lib().gcoo_static_handle_bytes(m, k, nnz, p))
    with _on(row_ptr.get_device()):
        if out_buf is None:
            if need == 0:
                raise GcooError(GCOO_ELIMIT if nnz > GCOO_STATIC_MAX_NNZ else GCOO_EINVAL, "gcoo_static_handle_bytes")
            out_buf = _alloc(need, row_ptr.device)
        if stream is not None:
            _used_on(out_buf, stream)
        out = C.c_void_p()
        _check(lib().gcoo_from_csr_device_static(m, k, nnz, row_ptr.data_ptr(), col_idx.data_ptr(), vals.data_ptr(), p,
                                                 out_buf.data_ptr(), out_buf.numel(), _stream_ptr(stream), C.byref(out)),
               "gcoo_from_csr_device_static")
    A = GcooMatrix(out.value, out_buf)
    A._mk = (m, k)
    return A


def gcoo_dense_nnz(A: torch.Tensor, stream=None) -> int:
    assert A.is_cuda and A.dtype == torch.float32 and A.dim() == 2 and A.stride(1) == 1
    n = C.c_int64()
    with _on(A.get_device()):
        _check(lib().gcoo_dense_nnz(A.shape[0], A.shape[1], A.data_ptr(), A.stride(0), _stream_ptr(stream), C.byref(n)),
               "gcoo_dense_nnz")
    return n.value


def gcoo_from_dense(A: torch.Tensor, p: int, stream=None) -> GcooMatrix:
    """Algorithm 1 as the paper runs it: count, allocate by the count, fill."""
    if stream is None and A.is_cuda:
        got = (_calls or _module()).from_dense(A, p, _raw_stream(A.get_device()))
        if got is not None:
            return _matrix(got, tuple(A.shape), "gcoo_from_dense")
    assert A.is_cuda and A.dtype == torch.float32 and A.dim() == 2 and A.stride(1) == 1
    m, k = A.shape
    L, lda = lib(), A.stride(0)
    nbytes = L.gcoo_dense_count_bytes(m, k, p)
    if nbytes == 0:
        raise GcooError(GCOO_EINVAL, "gcoo_dense_count_bytes")
    with _on(A.get_device()):
        sp = _stream_ptr(stream)
        counts = _alloc(nbytes, A.device)
        if stream is not None:
            _used_on(counts, stream)
        n, out = C.c_int64(), C.c_void_p()
        _check(L.gcoo_dense_count(m, k, A.data_ptr(), lda, p, counts.data_ptr(), counts.numel(), sp, C.byref(n)), "gcoo_from_dense")
        buf = _alloc(L.gcoo_device_bytes(m, k, n.value, p), A.device)
        if stream is not None:
            _used_on(buf, stream)
        _check(L.gcoo_from_dense_counted(m, k, n.value, A.data_ptr(), lda, p, counts.data_ptr(), buf.data_ptr(), buf.numel(), sp,
                                         C.byref(out)), "gcoo_from_dense")
    return GcooMatrix(out.value, buf)


def gcoo_spdm(A: GcooMatrix, B: torch.Tensor, C_out: torch.Tensor | None = None, variant: int = VARIANT_AUTO,
              stream=None) -> torch.Tensor:
    """C = A x B on the current stream.  B: [k, N] fp32 device tensor with unit column stride."""
    if stream is None and B.is_cuda:
        m, k = A._mk or A.shape
        got = (_calls or _module()).spdm(A._h or A._address(), m, k, B, C_out, _raw_stream(B.get_device()), variant)
        if got is not None:
            if type(got) is int:
                raise GcooError(got, "gcoo_spdm")
            return got
    assert B.is_cuda and B.dtype is torch.float32 and B.dim() == 2
    m, k = A._mk or A.shape
    kb, N = B.shape
    ldb, cs = B.stride()
    assert kb == k and (cs == 1 or N <= 1)
    if C_out is None:
        C_out = torch.empty((m, N), dtype=torch.float32, device=B.device)
        if stream is not None:
            _used_on(C_out, stream)
    assert C_out.is_cuda and C_out.dtype is torch.float32 and C_out.shape == (m, N)
    if k <= 1:
        ldb = max(N, 1)
    ldc = C_out.stride(0) if m > 1 else max(N, 1)
    d = B.get_device()
    if d != torch.cuda.current_device():
        with torch.cuda.device(d):
            return gcoo_spdm(A, B, C_out, variant, stream)
    handle = A._h or A._address()
    if stream is None:
        sp = _raw_stream(d)
    else:
        sp = stream.cuda_stream
        _used_on(A.buf, stream)
    status = lib().gcoo_spdm_variant(handle, B.data_ptr(), ldb, N, C_out.data_ptr(), ldc, sp, variant)
    if status:
        raise GcooError(status, "gcoo_spdm")
    return C_out


def gcoo_spdm_pick(A: GcooMatrix, B: torch.Tensor, C_out: torch.Tensor) -> int:
    return int(lib().gcoo_spdm_pick(A.handle, B.data_ptr(), B.stride(0), B.shape[1], C_out.data_ptr(), C_out.stride(0)))


def gcoo_spdm_kernel(A: GcooMatrix, B: torch.Tensor, C_out: torch.Tensor, variant: int = VARIANT_AUTO) -> int:
    """The kernel (KERNEL_*) that gcoo_spdm() launches for these arguments, or the negative status it fails with."""
    return int(lib().gcoo_spdm_kernel(A.handle, B.data_ptr(), B.stride(0), B.shape[1], C_out.data_ptr(), C_out.stride(0), variant))


def gcoo_csr_spmm_baseline(m: int, k: int, row_ptr: torch.Tensor, col_idx: torch.Tensor, vals: torch.Tensor,
                           B: torch.Tensor, C_out: torch.Tensor | None = None, stream=None) -> torch.Tensor:
    """The plain CSR row-split SpMM kept for comparison (device tensors only)."""
    assert row_ptr.is_cuda and row_ptr.dtype == torch.int32 and col_idx.dtype == torch.int32 and vals.dtype == torch.float32
    assert B.is_cuda and B.dtype == torch.float32 and B.dim() == 2 and B.shape[0] == k and (B.stride(1) == 1 or B.shape[1] <= 1)
    N = B.shape[1]
    if C_out is None:
        C_out = torch.empty((m, N), dtype=torch.float32, device=B.device)
    ldb = B.stride(0) if B.shape[0] > 1 else max(N, 1)
    ldc = C_out.stride(0) if C_out.shape[0] > 1 else max(N, 1)
    with torch.cuda.device(B.device):
        _check(baseline_lib().gcoo_csr_spmm_baseline(m, k, row_ptr.data_ptr(), col_idx.data_ptr(), vals.data_ptr(), B.data_ptr(), ldb, N,
                                            C_out.data_ptr(), ldc, _stream_ptr(stream)), "gcoo_csr_spmm_baseline")
    return C_out


def gcoo_default_p(m: int, k: int, nnz: int, N: int) -> int:
    return int(lib().gcoo_default_p(m, k, nnz, N))


def gcoo_tune_p(m: int, k: int, row_ptr, col_idx, vals, B: torch.Tensor, candidates=(8, 16, 32, 38, 42, 48, 64), reps: int = 5,
                include_conversion: bool = False):
    """Times conversion + product for each group height and returns (best p, {p: ms}).

    The tuner the paper leaves as future work (Section 5), in its simplest form: the matrix and a
    B of the real width are needed, nothing is modelled.  With include_conversion the time of
    the conversion counts too (a matrix that is multiplied once)."""
    C_out = torch.empty((m, B.shape[1]), dtype=torch.float32, device=B.device)
    times = {}
    for p in candidates:
        A = gcoo_from_csr(m, k, row_ptr, col_idx, vals, p, device=B.device)
        holder = [A]

        def step():
            if include_conversion:
                holder[0].free()
                holder[0] = gcoo_from_csr(m, k, row_ptr, col_idx, vals, p, device=B.device)
            gcoo_spdm(holder[0], B, C_out)

        step()
        torch.cuda.synchronize()
        ts = []
        for _ in range(reps):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            step()
            e1.record()
            torch.cuda.synchronize()
            ts.append(e0.elapsed_time(e1))
        ts.sort()
        times[p] = ts[len(ts) // 2]
        holder[0].free()
    return min(times, key=times.get), times



def gcoo_set_share_policy(policy: int) -> None:
    _check(lib().gcoo_set_share_policy(policy), "gcoo_set_share_policy")
