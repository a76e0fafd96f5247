"""The whole step (the conversion that allocates nothing + the product) recorded into a HIP graph and replayed:
gcoo_from_csr_device_static and gcoo_spdm launch kernels on the caller's stream and do nothing else, so a
stream capture can take them.  Every replay is checked against the same calls made eagerly, with the program's
own eager work and synchronisations between the replays, on inputs that change from replay to replay."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding, workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _step(L, w, p, dev, buf, B, Cout, variant, stream_ptr):
    h = C.c_void_p()
    rc = L.gcoo_from_csr_device_static(w.m, w.k, w.nnz, dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(), p,
                                       buf.data_ptr(), buf.numel(), stream_ptr, C.byref(h))
    assert rc == 0, rc
    rc = L.gcoo_spdm_variant(h, B.data_ptr(), B.stride(0), B.shape[1], Cout.data_ptr(), Cout.stride(0), stream_ptr, variant)
    assert rc == 0, rc
    return h


@pytest.mark.parametrize("case", ["register", "shared", "few_items", "tall_groups", "run_schedule", "few_items_run_schedule"])
def test_conversion_and_product_in_a_graph(case):
    """"register", "few_items" and "tall_groups" work row by row, the "run_schedule" ones through the register kernel."""
    L = binding.lib()
    if case in ("register", "run_schedule"):
        w, p, variant = workloads.uniform_random(1500, 2000, 516, 0.97, seed=1), 32, binding.VARIANT_REG
    elif case == "shared":
        w, p, variant = workloads.uniform_random(1500, 2000, 512, 0.97, seed=2), 42, binding.VARIANT_SHARE
    elif case in ("few_items", "few_items_run_schedule"):
        w, p, variant = workloads.zipf_rows(600, 3000, 260, seed=3, row_max=2000), 32, binding.VARIANT_REG
    else:
        w, p, variant = workloads.uniform_random(900, 1200, 260, 0.95, seed=4), 128, binding.VARIANT_AUTO
    print(f"graph: {case} p={p} nnz={w.nnz}", flush=True)
    binding.gcoo_set_share_policy(binding.SHARE_ALWAYS if case == "shared" else binding.SHARE_NEVER if case.endswith("run_schedule") else binding.SHARE_AUTO)
    kernel = binding.KERNEL_SHARE if case == "shared" else binding.KERNEL_SCHED if case.endswith("run_schedule") else binding.KERNEL_ROWS
    try:
        dev = [torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)]
        B = torch.from_numpy(w.B).to(DEV)
        need = int(L.gcoo_static_handle_bytes(w.m, w.k, w.nnz, p))
        assert need > 0
        buf_g = torch.empty(need, dtype=torch.uint8, device=DEV)
        buf_e = torch.empty(need, dtype=torch.uint8, device=DEV)
        C_g = torch.empty((w.m, w.N), device=DEV)
        C_e = torch.empty((w.m, w.N), device=DEV)
        # once eagerly first: the library takes the address of its scratch and raises kernel limits on its first call
        sp = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        h = _step(L, w, p, dev, buf_e, B, C_e, variant, sp)
        assert L.gcoo_spdm_kernel(h, B.data_ptr(), w.N, w.N, C_e.data_ptr(), w.N, variant) == kernel
        L.gcoo_free(h)
        torch.cuda.synchronize()

        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            sp_c = C.c_void_p(torch.cuda.current_stream().cuda_stream)
            h_g = _step(L, w, p, dev, buf_g, B, C_g, variant, sp_c)
        vals0 = dev[2].clone()
        for replay in range(4):
            # new values of A and of B for this replay; the structure (and so every launch shape) stays
            dev[2].copy_(vals0 * (1.0 + 0.25 * replay))
            B.add_(0.5 * replay)
            C_g.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            C_e.fill_(float("nan"))
            h_e = _step(L, w, p, dev, buf_e, B, C_e, variant, sp)
            torch.cuda.synchronize()
            L.gcoo_free(h_e)
            assert torch.equal(C_g, C_e), f"replay {replay}"
            assert not torch.isnan(C_g).any()
            # eager work of the program between the replays
            (C_g.sum() + B.sum()).item()
        L.gcoo_free(h_g)
    finally:
        binding.gcoo_set_share_policy(binding.SHARE_AUTO)


def _band_structures(seed):
    """Two CSR structures of the same shape and entry count: rows of 62 to 90 entries, and the same with twelve rows of 3000 among them."""
    rng = np.random.default_rng(seed)
    m, k = 4000, 3600
    even, uneven = rng.integers(62, 91, m), rng.integers(55, 81, m)
    uneven[1000:1012] = 3000
    while (d := int(even.sum() - uneven.sum())) != 0:                    # (entries moved one by one to rows that have room)
        i = rng.integers(0, m, min(abs(d), m))
        if d > 0:
            np.add.at(uneven, i, uneven[i] < 3000)
        else:
            np.add.at(even, i, 1)
    out = []
    for lens in (even, uneven):
        cols = [np.sort(rng.choice(k, n, replace=False)).astype(np.int32) for n in lens]
        out.append((np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), np.concatenate(cols)))
    return m, k, out


@pytest.mark.parametrize("variant,p,N", [(binding.VARIANT_AUTO, 32, 2048), (binding.VARIANT_SHARE, 32, 260), (binding.VARIANT_AUTO, 64, 2047)])
def test_band_schedule_in_a_graph(variant, p, N):
    """The sixteen-wave kernel and its schedule, recorded once and replayed on matrices of even and of uneven rows in turn: whether there is a
    schedule is decided by the device, on each replay anew.  The launches stay the same."""
    L = binding.lib()
    m, k, structures = _band_structures(N)
    nnz = len(structures[0][1])
    rng = np.random.default_rng(p)
    dev = [torch.empty(m + 1, dtype=torch.int32, device=DEV), torch.empty(nnz, dtype=torch.int32, device=DEV), torch.empty(nnz, device=DEV)]

    def load(i, values):
        dev[0].copy_(torch.from_numpy(structures[i][0]))
        dev[1].copy_(torch.from_numpy(structures[i][1]))
        dev[2].copy_(torch.from_numpy(values))
    values = rng.standard_normal(nnz).astype(np.float32)
    Bh = rng.standard_normal((k, N)).astype(np.float32)
    B = torch.from_numpy(Bh).to(DEV)
    w = workloads.Workload("band", m, k, N, structures[0][0], structures[0][1], values, Bh)
    need = int(L.gcoo_static_handle_bytes(m, k, nnz, p))
    buf_g, buf_e = [torch.empty(need, dtype=torch.uint8, device=DEV) for _ in range(2)]
    C_g, C_e = [torch.empty((m, N), device=DEV) for _ in range(2)]
    load(0, values)
    sp = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    h = _step(L, w, p, dev, buf_e, B, C_e, variant, sp)
    assert L.gcoo_spdm_kernel(h, B.data_ptr(), N, N, C_e.data_ptr(), N, variant) == binding.KERNEL_BAND
    L.gcoo_free(h)
    torch.cuda.synchronize()
    print(f"graph: band schedule, variant={variant} p={p} N={N} nnz={nnz}", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        h_g = _step(L, w, p, dev, buf_g, B, C_g, variant, C.c_void_p(torch.cuda.current_stream().cuda_stream))
    for replay, i in enumerate([0, 1, 1, 0, 1, 0]):
        values = rng.standard_normal(nnz).astype(np.float32)
        load(i, values)
        C_g.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        C_e.fill_(float("nan"))
        L.gcoo_free(_step(L, w, p, dev, buf_e, B, C_e, variant, sp))
        torch.cuda.synchronize()
        assert torch.equal(C_g, C_e), replay
        r0, r1 = 900, 1100                                       # the long rows among them
        C64, D64 = orc.spdm_csr(k, N, *structures[i], values, Bh, r0, r1)
        err, bad = orc.max_scaled_error(C_g[r0:r1].cpu().numpy(), C64, D64)
        assert bad == 0 and err < 2e-6, (replay, err, bad)
        (C_g.sum() + B.sum()).item()
    L.gcoo_free(h_g)


@pytest.mark.parametrize("m,per_row", [(500, 7), (3000, 200)])
def test_host_csr_is_refused_while_recording(m, per_row):
    """A host CSR input on a stream that records (one that fits the library's pinned buffers and one that does not): refused, the recording
    goes on, and its replays are not disturbed by conversions of host inputs between them."""
    L, k, p = binding.lib(), 2000, 32
    w = workloads.uniform_random(m, k, 64, 1.0 - per_row / k, seed=m)
    arrays = (w.row_ptr.ctypes.data, w.col_idx.ctypes.data, w.vals.ctypes.data)
    B = torch.from_numpy(w.B).to(DEV)
    need = int(L.gcoo_device_bytes(w.m, w.k, w.nnz, p))
    buf = torch.empty(need, dtype=torch.uint8, device=DEV)
    A = binding.gcoo_from_csr(w.m, w.k, w.row_ptr, w.col_idx, w.vals, p, device=DEV)
    want = binding.gcoo_spdm(A, B)
    Cg = torch.empty_like(want)
    torch.cuda.synchronize()
    print(f"graph: host CSR refused, m={m} nnz={w.nnz}", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp = torch.cuda.current_stream().cuda_stream
        h = C.c_void_p()
        assert L.gcoo_from_csr(w.m, w.k, *arrays, 0, p, buf.data_ptr(), need, sp, C.byref(h)) == binding.GCOO_EHIP and not h.value
        binding.gcoo_spdm(A, B, Cg)
    for replay in range(3):
        Cg.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Cg, want), replay
        binding.gcoo_from_csr(w.m, w.k, w.row_ptr, w.col_idx, w.vals * np.float32(2.0), p, device=DEV)


def test_counts_are_refused_while_recording():
    """Calls that wait for a number from the device, on a stream that records: refused, and the recording goes on without them."""
    L, p = binding.lib(), 32
    w = workloads.uniform_random(700, 900, 64, 0.97, seed=11)
    dev = [torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)]
    Ad = torch.zeros((w.m, w.k), device=DEV)
    Ad[torch.repeat_interleave(torch.arange(w.m, device=DEV), torch.diff(dev[0]).long()), dev[1].long()] = dev[2]
    B = torch.from_numpy(w.B).to(DEV)
    need = int(L.gcoo_device_bytes(w.m, w.k, w.nnz, p))
    buf = torch.empty(need, dtype=torch.uint8, device=DEV)
    A = binding.gcoo_from_dense(Ad, p)
    want = binding.gcoo_spdm(A, B)
    Cg = torch.empty_like(want)
    torch.cuda.synchronize()
    print("graph: counts refused", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp = torch.cuda.current_stream().cuda_stream
        h, n = C.c_void_p(), C.c_int64()
        got = [L.gcoo_from_csr(w.m, w.k, *[x.data_ptr() for x in dev], 1, p, buf.data_ptr(), need, sp, C.byref(h)),
               L.gcoo_dense_nnz(w.m, w.k, Ad.data_ptr(), w.k, sp, C.byref(n)),
               L.gcoo_from_dense(w.m, w.k, Ad.data_ptr(), w.k, p, buf.data_ptr(), need, sp, C.byref(h))]
        binding.gcoo_spdm(A, B, Cg)
    assert got == [binding.GCOO_EHIP] * 3 and not h.value
    for replay in range(3):
        Cg.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Cg, want), replay
        assert binding.gcoo_dense_nnz(Ad) == w.nnz
