"""The host code of libgcoo.so run without a GPU, on the HIP calls of tests/host/hip_on_host.cpp: which kernels a call launches, where it
waits, what it does when a HIP call fails.  Every case runs in a process of its own (`python -m tests.host_calls NAME`), which
loads no torch: its HIP runtime would be found before the one of the test."""
import ctypes as C
import os
import subprocess
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "host", "hip_on_host.cpp")
STUB = os.path.join(ROOT, "paper_2005_14469_amd", "_build", "libhip_on_host.so")
LIB = os.environ.get("GCOO_LIBRARY") or os.path.join(ROOT, "paper_2005_14469_amd", "libgcoo.so")
OK, EINVAL, ENOMEM, EHIP = 0, -1, -3, -4
AUTO, LDS, REG, SHARE = 0, 1, 2, 3


def build():
    os.makedirs(os.path.dirname(STUB), exist_ok=True)
    tmp = f"{STUB}.{os.getpid()}"
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", SOURCE, "-o", tmp])
    os.replace(tmp, STUB)


class Host:
    """The library on the host's HIP calls, and addresses for what it only passes on."""

    def __init__(self):
        self.hip = C.CDLL(STUB, mode=C.RTLD_GLOBAL)
        self.hip.host_set.argtypes = [C.c_char_p, C.c_longlong]
        self.hip.host_log.restype = C.c_char_p
        self.hip.host_told.restype = C.c_void_p
        self.hip.host_poke.argtypes = [C.c_char_p, C.c_void_p, C.c_int32]
        self.hip.host_starts.restype = C.POINTER(C.c_int32)
        self.L = C.CDLL(LIB)
        i64, i32, vp, sz = C.c_int64, C.c_int32, C.c_void_p, C.c_size_t
        for name, res, args in [
                ("gcoo_device_bytes", sz, [i64, i64, i64, i32]), ("gcoo_default_p", i32, [i64] * 4),
                ("gcoo_from_csr", C.c_int, [i64, i64, vp, vp, vp, C.c_int, i32, vp, sz, vp, C.POINTER(vp)]),
                ("gcoo_from_csr_device", C.c_int, [i64, i64, i64, vp, vp, vp, i32, vp, sz, vp, C.POINTER(vp)]),
                ("gcoo_dense_nnz", C.c_int, [i64, i64, vp, i64, vp, C.POINTER(i64)]),
                ("gcoo_dense_count_bytes", sz, [i64, i64, i32]),
                ("gcoo_dense_count", C.c_int, [i64, i64, vp, i64, i32, vp, sz, vp, C.POINTER(i64)]),
                ("gcoo_from_dense", C.c_int, [i64, i64, vp, i64, i32, vp, sz, vp, C.POINTER(vp)]),
                ("gcoo_from_dense_counted", C.c_int, [i64, i64, i64, vp, i64, i32, vp, vp, sz, vp, C.POINTER(vp)]),
                ("gcoo_spdm_variant", C.c_int, [vp, vp, i64, i64, vp, i64, vp, C.c_int]),
                ("gcoo_spdm_pick", C.c_int, [vp, vp, i64, i64, vp, i64]),
                ("gcoo_spdm_kernel", C.c_int, [vp, vp, i64, i64, vp, i64, C.c_int]),
                ("gcoo_free", C.c_int, [vp]), ("gcoo_set_share_policy", C.c_int, [C.c_int])]:
            f = getattr(self.L, name)
            f.restype, f.argtypes = res, args
        self.keep = []
        self.log()

    def set(self, key, value):
        self.hip.host_set(key.encode(), value)

    def log(self):
        return self.hip.host_log().decode().split("\n")[:-1]

    def launches(self):
        return [line.split()[1] for line in self.log() if line.startswith("launch")]

    def buffer(self, nbytes):
        """`nbytes` of memory at a multiple of 4096; kept."""
        raw = np.zeros(nbytes + 4096, np.uint8)
        self.keep.append(raw)
        return raw.ctypes.data + (-raw.ctypes.data) % 4096

    def matrix(self, m, k, nnz, p):
        """A handle of a CSR matrix on the device; no kernel looks at the arrays."""
        h = C.c_void_p()
        # (the conversion only launches: a place that nothing reads serves as the buffer, however large)
        rc = self.L.gcoo_from_csr_device(m, k, nnz, 1 << 20, 1 << 20, 1 << 20, p, 1 << 20, 1 << 50, None, C.byref(h))
        assert rc == OK, rc
        return h

    def spdm(self, h, N, ldb, variant=AUTO, ldc=None, B=1 << 30, Cp=1 << 40):
        return self.L.gcoo_spdm_variant(h, B, ldb, N, Cp, N if ldc is None else ldc, None, variant)


# ---- a row pitch of B of 2^30 elements or more ---------------------------------------------------

def wide_pitch(host):
    """The automatic choice serves any row pitch of B; the kernels that hold it in 32 bits refuse it when asked for."""
    for m, k, nnz, p in [(100, 2, 150, 32), (100, 2, 150, 128), (4000, 4000, 800000, 32), (8000, 8000, 320000, 42)]:
        h = host.matrix(m, k, nnz, p)
        for N in (1, 3, 4, 64, 513):
            for ldb in (1 << 30, (1 << 30) + 1, 1 << 33):
                host.log()
                assert host.spdm(h, N, ldb) == OK, (m, p, N, ldb)
                names = host.launches()
                assert len(names) == 1 and "spdm_lds" in names[0], (m, p, N, ldb, names)
                assert host.spdm(h, N, ldb, REG) == EINVAL and host.spdm(h, N, ldb, SHARE) == EINVAL
            host.log()
            assert host.spdm(h, N, (1 << 30) - 1) == OK
            assert "spdm_lds" not in host.launches()[0]


# ---- one to three columns, with a run schedule ----------------------------------------------------

def few_columns(host):
    """The automatic choice serves one to three columns whatever schedules the matrix carries."""
    for policy in (0, 1, 2):
        assert host.L.gcoo_set_share_policy(policy) == OK
        for m, k, nnz, p in [(40000, 5000, 3000000, 32), (70000, 5000, 9000000, 64), (70000, 300, 9000000, 100), (100, 200, 9000, 32)]:
            h = host.matrix(m, k, nnz, p)
            for N in (1, 2, 3, 4, 5):
                assert host.spdm(h, N, N) == OK, (policy, m, p, N)


# ---- calls that cannot be recorded ----------------------------------------------------------------

def _host_csr(host, m, k, per_row, p=32):
    """gcoo_from_csr() with arrays in host memory; the status."""
    rp = (np.arange(m + 1) * per_row).astype(np.int32)
    ci = np.tile(np.arange(per_row, dtype=np.int32), m)
    va = np.ones(m * per_row, np.float32)
    need = host.L.gcoo_device_bytes(m, k, m * per_row, p)
    h = C.c_void_p()
    rc = host.L.gcoo_from_csr(m, k, rp.ctypes.data, ci.ctypes.data, va.ctypes.data, 0, p, host.buffer(need), need, None, C.byref(h))
    assert bool(h.value) == (rc == OK)
    if rc == OK:
        host.L.gcoo_free(h)
    return rc


def host_csr_under_capture(host):
    """A host CSR input on a stream that records: refused, and nothing of it recorded - a replay would read the library's pinned
    buffer with whatever a later conversion has put there."""
    for m, k, per_row, p in [(500, 700, 7, 32), (500, 700, 7, 128), (40, 60000, 3, 32), (3000, 2000, 200, 32)]:
        assert _host_csr(host, m, k, per_row, p) == OK                        # (the pinned buffer is there)
        host.log()
        host.set("capturing", 1)
        assert _host_csr(host, m, k, per_row, p) == EHIP
        assert host.log() == []
        host.set("capturing", 0)
        assert _host_csr(host, m, k, per_row, p) == OK
        host.set("hipStreamIsCapturing", 1)                                  # (the default stream while another one records)
        assert _host_csr(host, m, k, per_row, p) == EHIP
        host.set("hipStreamIsCapturing", 0)


def counts_under_capture(host):
    """A call that waits for a number from the device, on a stream that records: refused, and nothing of it recorded - a replay would
    write its number where another call waits for its own."""
    m, k, p = 300, 500, 32
    n, h = C.c_int64(), C.c_void_p()
    buf = host.buffer(1 << 20)
    calls = [lambda: host.L.gcoo_from_csr(m, k, buf, buf, buf, 1, p, 1 << 20, 1 << 50, None, C.byref(h)),
             lambda: host.L.gcoo_dense_nnz(m, k, 1 << 20, k, None, C.byref(n)),
             lambda: host.L.gcoo_dense_count(m, k, 1 << 20, k, p, 1 << 20, 1 << 50, None, C.byref(n)),
             lambda: host.L.gcoo_from_dense(m, k, 1 << 20, k, p, 1 << 20, 1 << 50, None, C.byref(h))]
    host.set("answer", 1234)
    for call in calls:
        assert call() == OK
        host.log()
        host.set("capturing", 1)
        host.set("hipStreamSynchronize", 900)
        assert call() == EHIP
        assert host.log() == []
        host.set("capturing", 0)
        host.set("hipStreamSynchronize", 0)
        assert call() == OK


# ---- the pinned buffers of host inputs ---------------------------------------------------------------

def stage_release_fails(host):
    """The event behind the readers of a pinned buffer cannot be recorded: the call waits for the device before it gives the buffer
    back, and does not give it back at all where that fails too - its readers may still be queued."""
    shape = (500, 700, 7)
    assert _host_csr(host, *shape) == OK
    host.log()
    host.set("hipEventRecord", 1)
    assert _host_csr(host, *shape) == EHIP
    log = [line for line in host.log() if not line.startswith("launch")]
    assert log == ["record", "wait device"], log
    host.set("hipDeviceSynchronize", 1)
    for _ in range(4):                                                       # all four are lost
        assert _host_csr(host, *shape) == EHIP
    host.set("hipEventRecord", 0)
    host.set("hipDeviceSynchronize", 0)
    host.log()
    assert _host_csr(host, *shape) == OK
    log = host.log()
    assert "record" not in log and log.count("copy") == 3 and "wait stream" in log, log


def starts_of_a_changing_input(host):
    """Where the groups begin goes to the device in a launch's arguments, and the kernel reads and writes from there to there: whatever another thread does to the caller's arrays behind their check, no group begins or ends
    outside the entries, and once the arrays are copied nothing of them is read again."""
    m, k, per_row, p = 100, 200, 5, 32
    rp = (np.arange(m + 1) * per_row).astype(np.int32)
    ci, va = np.tile(np.arange(per_row, dtype=np.int32), m), np.ones(m * per_row, np.float32)
    need = host.L.gcoo_device_bytes(m, k, m * per_row, p)
    want = [0, 160, 320, 480, 500]
    for call, at, value, starts in [(b"", 0, 0, want), (b"hipHostGetDevicePointer", 64, 1 << 30, want), (b"hipHostGetDevicePointer", 100, 1 << 30, want),
                                    (b"hipStreamIsCapturing", 64, 1 << 30, [0, 160, 500, 480, 500]), (b"hipStreamIsCapturing", 32, -7, [0, 0, 320, 480, 500])]:
        mine, h = rp.copy(), C.c_void_p()
        if call:
            host.hip.host_poke(call, mine.ctypes.data + 4 * at, value)
        host.log()
        assert host.L.gcoo_from_csr(m, k, mine.ctypes.data, ci.ctypes.data, va.ctypes.data, 0, p, host.buffer(need), need, None, C.byref(h)) == OK
        assert any("order_groups_host" in name for name in host.launches())
        assert not call or mine[at] == value
        assert list(host.hip.host_starts()[:5]) == starts, (call, at, list(host.hip.host_starts()[:5]))
        host.L.gcoo_free(h)


def pinned_memory_is_coherent(host):
    """Memory that kernels read anew after the host has written to it, or write to under the host's eyes, is coherent by request, not by the process's default."""
    COHERENT = 0x40000000                                                    # hipHostMallocCoherent
    assert _host_csr(host, 500, 700, 7) == OK
    host.set("answer", 7)
    n = C.c_int64()
    assert host.L.gcoo_dense_nnz(30, 50, 1 << 20, 50, None, C.byref(n)) == OK
    flags = [int(line.split()[1]) for line in host.log() if line.startswith("pinned")]
    assert len(flags) == 2 and all(f & COHERENT for f in flags), flags


def slot_wait_fails(host):
    """The wait for a kernel that tells the host a number fails: nobody gets its slot again, the kernel may still write there.  With all slots lost such
    calls fail instead of waiting for one."""
    n = C.c_int64()
    host.set("answer", 77)
    host.set("hipStreamSynchronize", 1)
    places = set()
    for i in range(64):
        assert host.L.gcoo_dense_nnz(30, 50, 1 << 20, 50, None, C.byref(n)) == EHIP
        places.add(host.hip.host_told())
        if i == 3:                                                           # the other calls go on
            host.set("hipStreamSynchronize", 0)
            assert host.L.gcoo_dense_nnz(30, 50, 1 << 20, 50, None, C.byref(n)) == OK and n.value == 77
            assert host.hip.host_told() not in places
            host.set("hipStreamSynchronize", 1)
    assert len(places) == 64
    host.set("hipStreamSynchronize", 0)
    host.log()
    assert host.L.gcoo_dense_nnz(30, 50, 1 << 20, 50, None, C.byref(n)) == EHIP
    assert host.log() == []


def slot_launch_fails(host):
    """An error that an earlier call of the thread has left is reported behind a launch that went well: the kernel still tells its number, so its slot is
    given back behind it, and not at all where the wait for it fails."""
    m, k, dev = 300, 700, 1 << 20
    n, h = C.c_int64(), C.c_void_p()
    calls = [lambda: host.L.gcoo_from_csr(m, k, dev, dev, dev, 1, 8, 1 << 30, 1 << 50, None, C.byref(h)),
             lambda: host.L.gcoo_dense_nnz(m, k, dev, k, None, C.byref(n)),
             lambda: host.L.gcoo_dense_count(m, k, dev, k, 8, dev, 1 << 50, None, C.byref(n)),
             lambda: host.L.gcoo_from_dense(m, k, dev, k, 8, dev, 1 << 50, None, C.byref(h))]
    host.set("answer", 5)
    for call in calls:
        assert call() == OK
        free = host.hip.host_told()
        host.set("hipGetLastError", 1)
        host.log()
        assert call() == EHIP
        log = host.log()
        assert len(log) == 2 and log[0].startswith("launch") and log[1] == "wait stream", log
        assert host.hip.host_told() == free                                  # given back
        host.set("hipStreamSynchronize", 1)
        assert call() == EHIP and host.hip.host_told() == free
        host.set("hipGetLastError", 0)
        host.set("hipStreamSynchronize", 0)
        assert call() == OK and host.hip.host_told() != free                 # lost


def looks_before_waiting(host):
    """A conversion that goes on behind its counting kernel takes the number as soon as it is there and waits for the stream only where it does not
    come; a wait that fails is reported, and a stream that ended without a number is not taken for one."""
    m, k, nnz, dev = 300, 700, 1234, 1 << 20
    calls = [lambda n, h: host.L.gcoo_from_csr(m, k, dev, dev, dev, 1, 8, 1 << 30, 1 << 50, None, C.byref(h)),
             lambda n, h: host.L.gcoo_dense_count(m, k, dev, k, 8, dev, 1 << 50, None, C.byref(n))]
    for call in calls:
        n, h = C.c_int64(), C.c_void_p()
        host.set("answer", nnz)
        host.log()
        assert call(n, h) == OK and "wait stream" not in host.log()
        assert h.value if call is calls[0] else n.value == nnz
        host.set("answer", -1)
        assert call(n, h) not in (OK, EHIP) and host.log().count("wait stream") == 1
        host.set("hipStreamSynchronize", 1)
        assert call(n, h) == EHIP
        host.set("hipStreamSynchronize", 0)


# ---- where a dense conversion waits ------------------------------------------------------------------

def dense_waits(host):
    """gcoo_from_dense_counted() waits for nothing, gcoo_from_dense() once, whatever the group height."""
    m, k, nnz = 3000, 700, 1234
    host.set("answer", nnz)
    for p in (1, 32, 64, 65, 128, 256):
        n, h = C.c_int64(), C.c_void_p()
        assert host.L.gcoo_dense_count(m, k, 1 << 20, k, p, 1 << 20, 1 << 50, None, C.byref(n)) == OK and n.value == nnz
        host.log()
        assert host.L.gcoo_from_dense_counted(m, k, nnz, 1 << 20, k, p, 1 << 20, 1 << 30, 1 << 50, None, C.byref(h)) == OK
        log = host.log()
        assert all(line.startswith("launch") for line in log), (p, log)
        assert host.L.gcoo_from_dense(m, k, 1 << 20, k, p, 1 << 30, 1 << 50, None, C.byref(h)) == OK
        assert [line for line in host.log() if not line.startswith("launch")] == ["wait stream"], p
    host.set("capturing", 1)                                                 # so the former can be recorded
    assert host.L.gcoo_from_dense_counted(m, k, nnz, 1 << 20, k, 128, 1 << 20, 1 << 30, 1 << 50, None, C.byref(h)) == OK


# ---- how many launches a dense matrix takes --------------------------------------------------------------

def dense_launches(host):
    """The one launch for a dense matrix's orders is for groups that have work for its threads: not where more workgroups than two to a compute unit have few columns or entries each, nor for narrow groups that are mostly
    filled; with a band schedule it stands for two launches and is taken there."""
    def names(m, k, nnz, p):
        h = C.c_void_p()
        host.log()
        assert host.L.gcoo_from_dense_counted(m, k, nnz, 1 << 20, k, p, 1 << 20, 1 << 30, 1 << 50, None, C.byref(h)) == OK
        log = host.launches()
        host.L.gcoo_free(h)
        kinds = [x for x in ("fill_dense_groups", "fill_dense_masked", "band_fill") if any(x in name for name in log)]
        assert len(kinds) == len(log) or kinds[0] == "fill_dense_masked", log
        return kinds
    one, two = ["fill_dense_groups"], ["fill_dense_masked"]
    for m, p in [(512 * 32, 32), (512 * 64, 64), (512 * 8, 8)]:
        assert names(m, 64, 20 * m, p) == one and names(m + 1, 64, 20 * m, p) == two, p
    for k, per_group, p, kinds in [(199, 1500, 32, two), (200, 1500, 32, one), (200, 999, 32, two), (200, 1000, 32, one), (300, 4000, 32, two)]:
        assert names(20000, k, 625 * per_group, p) == kinds, (k, per_group)
    for k, per_group, p, kinds in [(64, 64 * 24, 32, one), (64, 64 * 25, 32, two), (65, 65 * 25, 32, one), (65, 1900, 64, one), (65, 2100, 64, two), (300, 2100, 64, two), (301, 2100, 64, one), (256, 4100, 32, one)]:
        assert names(10 * p, k, 10 * per_group, p) == kinds, (k, per_group, p)
    for m, k, nnz, p in [(64000, 1000, 1280000, 32), (300000, 128, 3840000, 32), (4000, 4000, 320000, 32)]:
        assert names(m, k, nnz, p) == ["fill_dense_groups", "band_fill"], (m, k)


# ---- LDS of the conversion by masks ----------------------------------------------------------------------

def order_lds(host):
    """A place of a group's entries in LDS is eight bytes, value and row and column in a word: one launch converts groups of as many entries as 61 KB hold of them beside the masks, and asks for no more than it uses."""
    for m, k, per_group, p, launches in [(3200, 1000, 5350, 32, 1), (3200, 1000, 5450, 32, 2), (3200, 2300, 2500, 32, 1), (3200, 2300, 2580, 32, 2), (6400, 1000, 4000, 64, 1)]:
        host.log()
        host.L.gcoo_free(host.matrix(m, k, per_group * (m // p), p))
        log = [line.split() for line in host.log() if line.startswith("launch")]
        assert len(log) == launches, (k, per_group, log)
        if launches == 1:
            keys, words, threads = 1 << (k - 1).bit_length(), p // 32, int(log[0][3])
            held = (int(log[0][4]) - 4 * (keys * (words + 1) + 2 * min(keys, threads))) / 8
            assert held == int(held) and per_group < held <= 3 * (per_group + 1) // 2 + 67 and int(log[0][4]) <= 61 * 1024, (k, per_group, log)


# ---- long rows of a dense matrix --------------------------------------------------------------------------

def places_in_turns(host):
    """The long rows of a dense matrix that one launch converted are dealt to the XCDs that share a tile; not where every XCD has whole tiles; those of a matrix from CSR arrays are in places too, in their order, and those of two launches are counted."""
    def dense(m, k, nnz, p):
        h = C.c_void_p()
        assert host.L.gcoo_from_dense_counted(m, k, nnz, 1 << 20, k, p, 1 << 20, 1 << 30, 1 << 50, None, C.byref(h)) == OK
        return h
    for h, N, kind in [(dense(2000, 1800, 20000, 32), 64, 2), (dense(2000, 1800, 20000, 32), 420, 2), (dense(2000, 1800, 20000, 32), 512, 1), (host.matrix(2000, 1800, 20000, 32), 64, 1), (dense(60000, 1024, 61000, 32), 64, 0)]:
        host.log()
        assert host.spdm(h, N, N) == OK
        (name,) = host.launches()
        assert f"RowsLongE{kind}E" in name, (N, kind, name)


# ---- a matrix without columns --------------------------------------------------------------------------

def no_columns(host):
    """A of k = 0 columns: the product is all zeros, and some kernel writes them, also where the register variant is asked for."""
    for policy in (0, 1, 2):
        assert host.L.gcoo_set_share_policy(policy) == OK
        for p in (1, 32, 64, 65, 256):
            h = host.matrix(500, 0, 0, p)
            for N in (1, 2, 3, 4, 260):
                host.log()
                assert host.spdm(h, N, N, AUTO, None, None) == OK, (policy, p, N)
                assert len(host.launches()) == 1
                wide = N >= (2 if 38 < p <= 64 else 4)
                status = host.spdm(h, N, N, REG, None, None)
                assert status == OK if wide else status in (OK, EINVAL), (policy, p, N, status)
                assert len(host.launches()) == (status == OK)


# ---- which kernel runs --------------------------------------------------------------------------------

def kernel_of_product(host):
    """gcoo_spdm_kernel() names the kernel that gcoo_spdm_variant() launches, or the status it fails with."""
    kernels = {1: ("spdm_lds",), 2: ("spdm_sched",), 3: ("spdm_share",), 4: ("spdm_rows", "spdm_vectors"), 5: ("spdm_band",)}
    seen = set()
    shapes = [(256, 256, 0.1), (4000, 4000, 0.05), (1777, 2301, 0.03), (8000, 8000, 0.005), (8000, 8000, 0.1), (12001, 12001, 0.0005),
              (16384, 16384, 0.0032), (20, 8000, 0.01), (385, 3600, 0.02), (5, 0, 0.0), (40, 7, 0.0), (0, 5, 0.0), (40000, 40, 0.5)]
    for policy in (0, 1, 2):
        assert host.L.gcoo_set_share_policy(policy) == OK
        for m, k, density in shapes:
            for p in (1, 32, 38, 42, 48, 64, 65, 256):
                h = host.matrix(m, k, int(m * k * density), p)
                for N, pad, off in [(0, 0, 0), (1, 0, 0), (3, 1, 4), (4, 0, 0), (64, 0, 0), (255, 0, 0), (256, 4, 4), (1024, 0, 0), (1117, 0, 0),
                                    (8000, 0, 0), (8000, 8, 16), (64, 1 << 30, 0), (256, 600000, 0)]:
                    for variant in (-1, 0, 1, 2, 3, 4):
                        B, Cp, ldb = (1 << 30) + off, (1 << 40) + off, N + pad
                        host.log()
                        kernel = host.L.gcoo_spdm_kernel(h, B, ldb, N, Cp, N, variant)
                        assert host.log() == []
                        status = host.spdm(h, N, ldb, variant, None, B, Cp)
                        names = host.launches()
                        what = (policy, m, k, density, p, N, pad, off, variant, kernel, status, names)
                        if kernel <= 0:
                            assert status == kernel and names == [], what
                            assert kernel == EINVAL or m == 0 or N == 0, what
                        else:
                            assert status == OK and names and all(any(x in n for x in kernels[kernel]) for n in names), what
                        seen.add((variant, kernel))
                host.L.gcoo_free(h)
    assert {(0, x) for x in (1, 2, 4, 5)} | {(2, 2), (2, 4), (3, 3), (3, 5)} <= seen, seen
    assert host.L.gcoo_spdm_kernel(None, 1 << 20, 4, 4, 1 << 20, 4, 0) == EINVAL


# ---- the tile of B in LDS --------------------------------------------------------------------------

# (m, k, N, entries, whether the row-by-row product goes by a tile of B in LDS): what tests/test_gpu_tile.py multiplies, and the shapes beside the lines of the rule
TILES = [(2047, 63, 500, 90000, True), (1023, 400, 1031, 102300, True), (1024, 400, 1031, 102400, True), (500, 1000, 17, 200000, True), (4000, 1500, 31, 600000, True),
         (700, 1280, 48, 300000, True), (700, 1279, 1031, 300000, True), (100, 2496, 517, 90000, True), (7, 2558, 4000, 14000, True), (92, 2550, 1024, 90000, True),
         (93, 2550, 1024, 90000, True), (1777, 2301, 1117, 122666, True), (300, 1, 1031, 18000, True), (100, 2, 500, 20000, True), (2100, 4, 500, 42000, True), (4000, 6, 500, 24000, True), (1000, 10, 1000, 10000, True), (500, 14, 2000, 5600, True),
         (300, 14, 4000, 4200, True), (2100, 15, 500, 16800, True), (2100, 16, 500, 16800, True), (7, 2559, 4000, 14000, False), (500, 1000, 15, 200000, False), (256, 256, 256, 6553, False), (2500, 2500, 64, 62500, False)]


def tiles(host):
    for m, k, N, nnz, tile in TILES:
        for variant in (AUTO, REG):
            for ldb, off in ((N, 0), (N + 3, 4)):
                host.log()
                h = host.matrix(m, k, nnz, 32)
                host.log()
                assert host.spdm(h, N, ldb, variant, N + 5, (1 << 30) + off, (1 << 40) + off) == OK
                (line,) = [x for x in host.log() if x.startswith("launch")]
                assert ("spdm_rows_tile" in line) == tile, (m, k, N, nnz, variant, line)
                if tile:
                    # behind the tile and its row of zeros, and behind the 256 bins that lie there before: where the rows begin, and the rows in their order
                    workgroups, _, shared = (int(x) for x in line.split()[2:])
                    rows = -(-m // (workgroups // -(-N // 16)))                  # of a workgroup, at least
                    assert shared >= max(64 * (k + 1), 1024) + 4 * (rows + 1) + 2 * rows, (m, k, N, nnz, line)
        # a B that the buffer descriptor does not reach
        assert host.spdm(h, N, (1 << 32) // (4 * k) + N, AUTO) == OK and "spdm_rows_tile" not in host.launches()[0], (m, k, N)


# ---- the widths of a slot ------------------------------------------------------------------------------

# (lanes of a slot, rows of B in flight, sums of a row: the instance of the row-by-row kernel; m, k, N, entries of every row): what tests/test_gpu_rows.py compares bit by bit
SUMS = [(64, 16, 4, 333, 333, 333, 21), (64, 8, 4, 422, 422, 285, 15), (32, 16, 2, 9000, 9000, 85, 49), (32, 8, 2, 9000, 9000, 85, 13), (16, 16, 2, 5000, 5700, 27, 45), (8, 16, 1, 9000, 5700, 13, 45),
        (16, 16, 1, 9000, 9000, 64, 49)]


def sums(host):
    for lanes, ahead, parts, m, k, N, per_row in SUMS:
        h = host.matrix(m, k, m * per_row, 32)
        host.log()
        assert host.spdm(h, N, N) == OK
        (name,) = host.launches()
        assert f"spdm_rowsILi{lanes}ELb0ELi{ahead}ELi{parts}E" in name, (m, k, N, per_row, name)


# (m, k, N, entries of every row; lanes of a slot, workgroups)
WIDTHS = [(8123, 11104, 22, 13, 8, 254), (7000, 7000, 22, 30, 8, 219), (3200, 3000, 40, 20, 16, 200), (3100, 3000, 40, 20, 16, 194), (3000, 3000, 40, 20, 16, 750), (700, 600, 300, 11, 64, 350),
          (6133, 5725, 93, 108, 32, 767), (6133, 5725, 93, 64, 32, 767), (6133, 5725, 93, 63, 16, 768), (6133, 5725, 96, 108, 16, 768),
          (299, 300, 300, 28, 16, 375), (299, 300, 300, 27, 64, 150), (300, 300, 300, 28, 64, 150),
          (205, 300, 205, 74, 16, 208), (349, 300, 300, 36, 16, 440), (350, 300, 300, 36, 64, 175),
          (513, 600, 300, 36, 16, 645), (512, 600, 300, 36, 64, 256), (513, 600, 300, 35, 64, 258), (699, 700, 383, 36, 16, 264), (699, 700, 384, 36, 64, 350), (700, 700, 383, 36, 64, 350),
          (1200, 3000, 140, 60, 64, 300),
          (2600, 2500, 256, 5, 64, 650), (2600, 2501, 256, 5, 16, 652), (2600, 2501, 255, 5, 64, 650), (1600, 1500, 320, 5, 64, 800), (1600, 1501, 320, 5, 16, 500), (6000, 6000, 128, 12, 16, 750),
          (3218, 3218, 326, 93, 32, 1209), (3218, 3218, 321, 93, 32, 1209), (3218, 3218, 257, 93, 16, 1010), (3218, 3218, 319, 93, 16, 1010), (3218, 3218, 326, 63, 16, 1212), (3218, 3218, 320, 93, 16, 1010)]


def widths(host):
    """Which instance of the row-by-row kernel a launch takes, and how many rows a wave has."""
    for m, k, N, per_row, lanes, workgroups in WIDTHS:
        h = host.matrix(m, k, m * per_row, 32)
        host.log()
        assert host.spdm(h, N, N) == OK
        (line,) = [x for x in host.log() if x.startswith("launch")]
        got = int(line.split()[2])
        assert f"spdm_rowsILi{lanes}ELb0E" in line and workgroups <= got < workgroups + 8, (m, k, N, per_row, line)


# ---- the cuts of the band schedule -------------------------------------------------------------------

# (m, k, N, entries, variant): what tests/test_gpu_band.py multiplies by the wide cut and by the tall one, and by which instance (Lb1: requests within a band's first unit, below 20 entries of a (wave, band); in the wide
# cut it was below 28, four of these are between, and 522 matrices are faster so: requests())
CUTS = [("ILi2ELb0E", 384, 3500, 260, 384 * 150, SHARE), ("ILi2ELb0E", 777, 3500, 252, 777 * 150, SHARE), ("ILi4ELb0E", 4000, 4000, 2044, 320000, AUTO),
        ("ILi4ELb0E", 4000, 3000, 1001, 1200000, AUTO), ("ILi2ELb1E", 384, 3500, 260, 384 * 60, SHARE), ("ILi2ELb1E", 777, 3500, 252, 777 * 62, SHARE),
        ("ILi2ELb1E", 97, 3500, 64, 97 * 130, SHARE), ("ILi2ELb1E", 300, 7000, 1000, 9450, SHARE), ("ILi2ELb1E", 40, 3500, 256, 2800, SHARE),
        ("ILi2ELb0E", 5000, 5001, 2501, 125025, AUTO), ("ILi4ELb0E", 4000, 4000, 2045, 320000, AUTO), ("ILi2ELb1E", 5600, 5601, 2601, 90000, AUTO),
        ("ILi4ELb0E", 2600, 3500, 260, 2600 * 150, SHARE), ("ILi4ELb0E", 4607, 3500, 252, 4607 * 150, SHARE), ("ILi4ELb0E", 4700, 3500, 252, 4700 * 62, SHARE),
        ("ILi2ELb0E", 2700, 3500, 260, 2700 * 60, SHARE), ("ILi4ELb0E", 1500, 3500, 64, 1500 * 150, SHARE), ("ILi4ELb1E", 1000, 3500, 64, 1000 * 205, SHARE),
        ("ILi2ELb0E", 301, 2962, 2427, 301 * 350, AUTO), ("ILi2ELb0E", 120, 6000, 6000, 120 * 900, AUTO), ("ILi4ELb0E", 1836, 2885, 1836, 1836 * 577, AUTO)]


def cuts(host):
    for instance, m, k, N, nnz, variant in CUTS:
        h = host.matrix(m, k, nnz, 32)
        host.log()
        assert host.spdm(h, N, N, variant) == OK
        names = host.launches()
        assert len(names) == 1 and "spdm_band" + instance in names[0], (m, k, N, nnz, names)
    # the tall cut's heads hold a column and the distance to the next one in a word
    for k in (65536, 65537):
        h = host.matrix(60000, k, 60000 * 300, 32)
        host.log()
        assert host.spdm(h, 4096, 4096) == OK
        assert "spdm_bandILi%dE" % (2 if k == 65536 else 4) in host.launches()[0], k


def requests(host):
    """When the rows of the next band are asked for, by the entries of a (wave, band); in the wide cut the late half behind the second step of its first unit up to 20, behind that unit from there on
    (measured, us: 4000 x 4000, 2 %, 25 entries: 88.6 88.2; 8632 x 8488, 1.7 %, 24 entries: 730 715; the other way round at 17: 7417 x 7331, 1.2 %: 366 369)."""
    for m, k, N, nnz, kernel in [(1000, 3000, 2045, 150000, "ILi4ELb1ELb0E"), (7417, 7331, 7272, 631827, "ILi4ELb1ELb1E"), (4000, 4000, 2045, 224000, "ILi4ELb1ELb1E"), (4000, 4000, 4000, 320000, "ILi4ELb0ELb0E"),
                                 (4000, 4000, 2053, 480000, "ILi4ELb0ELb0E"), (4000, 4000, 2053, 640000, "ILi4ELb0ELb1E"), (5600, 5601, 2601, 90000, "ILi2ELb1ELb0E"), (5000, 5001, 2605, 210000, "ILi2ELb0ELb0E"),
                                 (5000, 5001, 2605, 235000, "ILi2ELb0ELb1E")]:
        h = host.matrix(m, k, nnz, 32)
        host.log()
        assert host.spdm(h, N, N) == OK
        (name,) = host.launches()
        assert "spdm_band" + kernel in name, (m, k, N, nnz, name)


def tall_rounds(host):
    """Where a (wave, band) has many entries a launch in the tall cut costs whole rounds of its workgroups over the 256 compute units: one that leaves much of its
    last round idle is not taken (measured, us, with the idle round and with the height taken: 9000 x 9000, 1 %: 776 657; 9600 x 9600, 0.9 %: 798 720; 10000 x 10000, 0.75 %:
    804 760; 10240 x 10240, 0.75 %: 804 721; 11000 x 11000, 0.75 %, the wide cut instead: 1028 1014)."""
    for n, density in [(9000, 0.01), (9600, 0.009), (10000, 0.0075), (10240, 0.0075), (11000, 0.0075)]:
        h = host.matrix(n, n, round(n * n * density), 32)
        host.log()
        assert host.spdm(h, n, n) == OK
        (line,) = [x for x in host.log() if x.startswith("launch")]
        workgroups = int(line.split()[2])
        assert workgroups >= 0.95 * 256 * -(-workgroups // 256), (n, density, line)


def parts_of_power_law_rows(host):
    """The groups of a matrix with thirteen columns per entry of a group, as 20000 power-law rows have (exponent 1.5, at most 4096 entries), are cut into five parts: with three,
    one workgroup had a third of a heavy group to itself (the conversion, us: 61 with three, 42 with five).  Where the bands are filled in the same launch parts are larger."""
    for m, k, nnz, parts in [(20000, 20000, 944083, 5), (17000, 20000, 822886, 5), (18000, 20000, 847083, 5), (20000, 20000, 980676, 5), (20000, 20000, 800000, 3)]:
        host.log()
        host.matrix(m, k, nnz, 32)
        (line,) = [x for x in host.log() if "order_groups" in x]
        assert int(line.split()[2]) == parts * ((m + 31) // 32), (m, k, nnz, line)
    host.matrix(14000, 14000, 470400, 32)
    assert any("order_and_fill" in x for x in host.log())


# ---- threads ---------------------------------------------------------------------------------------------

def one_handle_many_threads(host):
    """Eight threads multiply with one handle and convert matrices of their own beside it: every call launches what it launches
    alone, and nothing writes to the handle."""
    import threading
    libc = C.CDLL(None)
    libc.malloc_usable_size.restype, libc.malloc_usable_size.argtypes = C.c_size_t, [C.c_void_p]
    shape = (4000, 4000, 800000, 32)
    h = host.matrix(*shape)
    inside = C.string_at(h, libc.malloc_usable_size(h))
    host.log()
    calls = [(8000, AUTO), (64, AUTO), (1, AUTO), (260, REG), (512, SHARE), (100, LDS)]

    def work(wrong):
        for _ in range(50):
            for N, variant in calls:
                if host.spdm(h, N, N, variant) != OK:
                    wrong.append((N, variant))
            host.L.gcoo_free(host.matrix(*shape))
            if _host_csr(host, 500, 700, 7) != OK:
                wrong.append("host")

    def launched(threads):
        wrong = []
        ts = [threading.Thread(target=work, args=(wrong,)) for _ in range(threads)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert wrong == []
        return sorted(line for line in host.log() if line.startswith("launch"))

    alone = launched(1)
    assert launched(8) == sorted(alone * 8)
    assert C.string_at(h, libc.malloc_usable_size(h)) == inside


if __name__ == "__main__":
    globals()[sys.argv[1]](Host())
    print("ok")
