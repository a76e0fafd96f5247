"""Counting and filling a dense matrix where the split can go wrong: no rows or no columns, one block and many, more blocks than the
last workgroup scans at a time, 64 and 65 rows per group (a bit per element, and walking twice), columns in fours and one by one.
Both routes of the C interface, bit for bit against the CPU oracle."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("m,k,p,density", [(1, 1, 1, 1.0), (0, 8, 4, 0.0), (5, 0, 4, 0.0), (33, 1023, 32, 0.05), (130, 1024, 64, 0.3),
                                           (130, 1028, 65, 0.3), (63, 4097, 64, 0.02), (70, 260, 7, 0.0), (64, 512, 64, 1.0), (2100, 1500, 1, 0.1),
                                           (2100, 301, 1, 0.1)])
def test_counts_and_fill(m, k, p, density):
    print(f"dense count: {m}x{k} p={p}", flush=True)
    rng = np.random.default_rng(m + k)
    Ah = (rng.standard_normal((m, k)) * (rng.random((m, k)) < density)).astype(np.float32)
    if m * k > 4:
        Ah[-1, -1] = np.nan
        Ah[0, 0] = -0.0
    A = torch.from_numpy(Ah).to(DEV)
    L, n = binding.lib(), C.c_int64()
    stream = torch.cuda.current_stream().cuda_stream
    assert L.gcoo_dense_nnz(m, k, A.data_ptr(), k, stream, C.byref(n)) == 0
    if m and k:
        want = orc.gcoo_from_dense(Ah, p)
        assert n.value == want.nnz
    handles = [binding.gcoo_from_dense(A, p)] if m and k else []
    buf = torch.empty(max(256, L.gcoo_device_bytes(m, k, n.value, p)), dtype=torch.uint8, device=DEV)
    out = C.c_void_p()
    assert L.gcoo_from_dense(m, k, A.data_ptr(), k, p, buf.data_ptr(), buf.numel(), stream, C.byref(out)) == 0
    handles.append(binding.GcooMatrix(out.value, buf))
    for h in handles:
        e = h.export()
        if m and k:
            assert np.array_equal(e["values"].view(np.uint32), want.values.view(np.uint32))
            assert np.array_equal(e["rows"], want.rows) and np.array_equal(e["cols"], want.cols)
            assert np.array_equal(e["gIdxes"], want.gIdxes) and np.array_equal(e["nnzPerGroup"], want.nnzPerGroup)
        else:
            assert len(e["values"]) == 0 and not e["gIdxes"].any()


@pytest.mark.parametrize("p", [7, 8, 9, 31, 32, 63, 64, 65])
@pytest.mark.parametrize("k,density", [(511, 1.0), (512, 1.0), (513, 0.6), (1024, 0.5), (1025, 0.02), (4100, 0.02), (4608, 1.0), (5121, 0.6)])
def test_fill_from_the_masks_of_the_count(p, k, density):
    """8 to 64 rows per group are filled from a bit per element that the count left in its buffer, other heights and a count in the matrix's
    own buffer by reading the matrix again: both against the oracle, rows that are longer than k, columns in fours and one by one, blocks of less than a list, of a
    whole one (8 x 512 entries) and of many, with and without an entry in the last row of a group; up to 4096 columns the bits are those of a group, beyond of a block of columns."""
    print(f"dense fill: k={k} p={p} density={density}", flush=True)
    rng = np.random.default_rng(k + p)
    m = 2 * p + 3
    Ah = (rng.standard_normal((m, k)) * (rng.random((m, k)) < density)).astype(np.float32)
    Ah[p - 1] = 0.0
    L, stream = binding.lib(), torch.cuda.current_stream().cuda_stream
    for pitch, off in ((k + (-k % 4) + 4, 0), (k + 3, 1)):
        whole = torch.full((m * pitch + off,), 7.0, device=DEV)
        A = whole[off:].view(m, pitch)[:, :k]
        A.copy_(torch.from_numpy(Ah))
        want = orc.gcoo_from_dense(Ah, p)
        handles = [binding.gcoo_from_dense(A, p)]
        buf = torch.empty(L.gcoo_device_bytes(m, k, want.nnz, p), dtype=torch.uint8, device=DEV)
        out = C.c_void_p()
        assert L.gcoo_from_dense(m, k, A.data_ptr(), pitch, p, buf.data_ptr(), buf.numel(), stream, C.byref(out)) == 0
        handles.append(binding.GcooMatrix(out.value, buf))
        for h in handles:
            e = h.export()
            assert np.array_equal(e["values"].view(np.uint32), want.values.view(np.uint32))
            assert np.array_equal(e["rows"], want.rows) and np.array_equal(e["cols"], want.cols)
            assert np.array_equal(e["gIdxes"], want.gIdxes) and np.array_equal(e["nnzPerGroup"], want.nnzPerGroup)


@pytest.mark.parametrize("workgroups", [1, 2, 31, 32, 33, 63, 65, 1023, 1024, 1025, 2500])
def test_arrivals_of_few_and_many_workgroups(workgroups):
    """The workgroups of a counting launch arrive at up to 32 words, which are zero again behind it: counts and offsets of launches with fewer
    workgroups than words, one more, and more pieces than workgroups, several times over."""
    print(f"dense count: {workgroups} pieces", flush=True)
    rng = np.random.default_rng(workgroups)
    Ah = (rng.random((16 * workgroups, 8)) < 0.3).astype(np.float32)
    A, few = torch.from_numpy(Ah).to(DEV), torch.from_numpy(Ah[:workgroups]).to(DEV)
    want = orc.gcoo_from_dense(Ah[:workgroups], 1)
    for _ in range(3):
        assert binding.gcoo_dense_nnz(A) == np.count_nonzero(Ah)
        e = binding.gcoo_from_dense(few, 1).export()
        assert np.array_equal(e["gIdxes"], want.gIdxes) and np.array_equal(e["nnzPerGroup"], want.nnzPerGroup)
        assert np.array_equal(e["rows"], want.rows) and np.array_equal(e["cols"], want.cols)


@pytest.mark.parametrize("copies", [0, 4, 200])
def test_counts_come_from_streams_at_rest_and_at_work(copies):
    """The conversions that need a count look for it a while and then wait for their stream: with nothing before them, with a little and with more than
    they look for (64 MB copies), on two streams in turn, the matrix written anew on the stream before each."""
    print(f"counts behind {copies} copies", flush=True)
    rng = np.random.default_rng(copies)
    n = 900
    Ah = (rng.standard_normal((n, n)) * (rng.random((n, n)) < 0.05)).astype(np.float32)
    want = orc.gcoo_from_dense(Ah, 32)
    r, c = np.nonzero(Ah)
    src = [torch.from_numpy(x).to(DEV) for x in (Ah, np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int32),
                                                 c.astype(np.int32), Ah[r, c])]
    big, x = torch.randn((4096, 4096), device=DEV), torch.empty((4096, 4096), device=DEV)
    streams = [torch.cuda.Stream(device=DEV) for _ in range(2)]
    torch.cuda.synchronize()
    exports = []
    for i in range(8):
        st = streams[i % 2]
        with torch.cuda.stream(st):
            A, row_ptr, cols, vals = [torch.zeros_like(t) for t in src]
            for _ in range(copies):
                x.copy_(big)
            for to, t in zip((A, row_ptr, cols, vals), src):
                to.copy_(t)
            H = binding.gcoo_from_dense(A, 32) if i % 4 < 2 else binding.gcoo_from_csr(n, n, row_ptr, cols, vals, 32, device=DEV)
            exports.append(H.export())
        torch.cuda.synchronize()
    for e in exports:
        assert np.array_equal(e["values"].view(np.uint32), want.values.view(np.uint32))
        assert np.array_equal(e["rows"], want.rows) and np.array_equal(e["cols"], want.cols) and np.array_equal(e["gIdxes"], want.gIdxes)


@pytest.mark.parametrize("m,k,p", [(700, 900, 65), (130, 1031, 128), (3000, 260, 256)])
def test_fill_of_tall_groups_in_a_graph(m, k, p):
    """gcoo_from_dense_counted() waits for nothing and can be recorded, for groups of more than 64 rows too, whose regrouped copy is counted
    on the device alone.  Replayed on new values in the same cells, against the oracle."""
    print(f"dense count: {m}x{k} p={p} in a graph", flush=True)
    rng = np.random.default_rng(p)
    Ah = (rng.standard_normal((m, k)) * (rng.random((m, k)) < 0.07)).astype(np.float32)
    A, B = torch.from_numpy(Ah).to(DEV), torch.from_numpy(rng.standard_normal((k, 68)).astype(np.float32)).to(DEV)
    L, n, h = binding.lib(), C.c_int64(), C.c_void_p()
    counts = torch.empty(L.gcoo_dense_count_bytes(m, k, p), dtype=torch.uint8, device=DEV)
    sp = torch.cuda.current_stream().cuda_stream
    assert L.gcoo_dense_count(m, k, A.data_ptr(), k, p, counts.data_ptr(), counts.numel(), sp, C.byref(n)) == 0
    need = L.gcoo_device_bytes(m, k, n.value, p)
    buf = torch.full((need,), 0x5a, dtype=torch.uint8, device=DEV)
    Cg = torch.empty((m, 68), device=DEV)
    binding.gcoo_spdm(binding.gcoo_from_dense(A, p), B, Cg)                # (kernel limits are raised on a first call)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp = torch.cuda.current_stream().cuda_stream
        assert L.gcoo_from_dense_counted(m, k, n.value, A.data_ptr(), k, p, counts.data_ptr(), buf.data_ptr(), need, sp, C.byref(h)) == 0
        H = binding.GcooMatrix(h.value, buf)
        binding.gcoo_spdm(H, B, Cg)
    for replay in range(4):
        A.mul_(1.25)
        Cg.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        want = orc.gcoo_from_dense(A.cpu().numpy(), p)
        e = H.export()
        assert np.array_equal(e["values"].view(np.uint32), want.values.view(np.uint32)) and np.array_equal(e["rows"], want.rows)
        assert np.array_equal(e["cols"], want.cols) and np.array_equal(e["gIdxes"], want.gIdxes)
        Ce = binding.gcoo_spdm(binding.gcoo_from_dense(A, p), B)
        assert torch.equal(Cg, Ce), replay
        ref = A.double() @ B.double()
        assert ((Cg.double() - ref).abs().max() / ref.abs().max()).item() < 2e-6


@pytest.mark.parametrize("m,k,p,density,long_rows", [
    (70, 255, 32, 0.3, 0), (69, 256, 32, 0.9, 1), (40, 300, 8, 0.2, 1), (130, 513, 31, 1.0, 0),
    (130, 4095, 31, 0.02, 1), (130, 4096, 32, 0.029, 0), (130, 4096, 32, 0.031, 2), (130, 4097, 32, 0.02, 1), (100, 2000, 33, 0.03, 1), (100, 2000, 64, 0.02, 0), (67, 4096, 64, 0.5, 0),
    (2100, 2600, 32, 0.05, 0), (2113, 2600, 31, 0.05, 3), (2100, 2500, 40, 0.08, 70), (1500, 4096, 64, 0.03, 5), (1501, 2900, 9, 0.06, 0)])
def test_row_order_and_bands_of_a_dense_matrix(m, k, p, density, long_rows):
    """The order by rows, the rows that are long and the columns of the bands come with the fill where the count left its masks, up to 4096 columns: one, two and four workgroups to a group, entries that fit
    the LDS and that do not, groups across two blocks of the band schedule, rows many times as long as the others, few and so many together that no bands are built.  Whole numbers, so that the
    product is exact: by rows and, the widest of a matrix of some size, by the band schedule."""
    print(f"dense rows and bands: {m}x{k} p={p} density={density} long={long_rows}", flush=True)
    rng = np.random.default_rng(m + k + p)
    Ah = (rng.integers(1, 8, (m, k)) * (rng.random((m, k)) < density)).astype(np.float32)
    Ah[rng.integers(0, m, 3)] = 0.0
    at = m // 2
    Ah[at:at + long_rows] = rng.integers(1, 8, (min(long_rows, m - at), k))
    A = torch.from_numpy(Ah).to(DEV)
    B = torch.from_numpy(rng.integers(-8, 8, (k, 2504)).astype(np.float32)).to(DEV)
    want = torch.from_numpy(Ah.astype(np.float64) @ B.cpu().numpy().astype(np.float64)).to(DEV)
    e, ref = binding.gcoo_from_dense(A, p).export(), orc.gcoo_from_dense(Ah, p)
    assert np.array_equal(e["values"], ref.values) and np.array_equal(e["rows"], ref.rows) and np.array_equal(e["cols"], ref.cols)
    for _ in range(2):
        H = binding.gcoo_from_dense(A, p)
        for N in (8, 64, 2504):
            C = torch.full((m, N), 7.0, device=DEV)
            kernel = binding.gcoo_spdm_kernel(H, B[:, :N], C)
            binding.gcoo_spdm(H, B[:, :N], C)
            assert torch.equal(C.double(), want[:, :N]), (N, kernel)
        assert kernel == binding.KERNEL_BAND or m < 1500


@pytest.mark.parametrize("long_rows", ["none", "last", "many"])
def test_more_lists_than_a_workgroup_looks_at(long_rows):
    """2672 lists of a dense matrix: none of them heavy, so that all have to be written; one in the last rows, which one workgroup finds; and one in about a hundred.  Whole numbers, so that the product is exact."""
    m, k, N = 64001, 1000, 2504
    print(f"dense, many lists: long={long_rows}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(7)
    share = torch.full((m, 1), 0.02, device=DEV)
    if long_rows == "last":
        share[-8:] = 0.9
    elif long_rows == "many":
        share.view(-1)[:m - 1].view(-1, 10)[::250] = 0.9
    A = torch.randint(1, 8, (m, k), generator=g, device=DEV, dtype=torch.float32) * (torch.rand((m, k), generator=g, device=DEV) < share)
    B = torch.randint(-8, 9, (k, N), generator=g, device=DEV, dtype=torch.float32)
    H = binding.gcoo_from_dense(A, 32)
    for cols in (64, N):
        C_ = torch.full((m, cols), 7.0, device=DEV)
        kernel = binding.gcoo_spdm_kernel(H, B[:, :cols], C_)
        binding.gcoo_spdm(H, B[:, :cols], C_)
        assert torch.equal(C_.double(), A.double() @ B[:, :cols].double()), (cols, kernel)
    assert kernel == binding.KERNEL_BAND


@pytest.mark.parametrize("m,k,p,density,long_rows", [(16417, 64, 32, 0.1, 3), (1025, 60, 64, 0.5, 0), (131, 64, 64, 1.0, 0), (130, 300, 64, 0.5, 1), (4200, 700, 8, 0.01, 2), (17000, 199, 32, 0.2, 0), (17000, 200, 32, 0.2, 0)])
def test_fill_and_order_by_rows_in_launches_of_their_own(m, k, p, density, long_rows):
    """Without bands: more groups than two to a compute unit with few columns or entries each, and narrow ones that are mostly filled; the last but one beside the last, where one launch does it."""
    print(f"dense, two launches: {m}x{k} p={p} density={density}", flush=True)
    rng = np.random.default_rng(m + k + p)
    Ah = (rng.integers(1, 8, (m, k)) * (rng.random((m, k)) < density)).astype(np.float32)
    Ah[m // 2:m // 2 + long_rows] = rng.integers(1, 8, (long_rows, k))
    A = torch.from_numpy(Ah).to(DEV)
    B = torch.from_numpy(rng.integers(-8, 8, (k, 130)).astype(np.float32)).to(DEV)
    H = binding.gcoo_from_dense(A, p)
    e, ref = H.export(), orc.gcoo_from_dense(Ah, p)
    assert np.array_equal(e["values"], ref.values) and np.array_equal(e["rows"], ref.rows) and np.array_equal(e["cols"], ref.cols)
    for N in (1, 4, 64, 130):
        C_ = binding.gcoo_spdm(H, B[:, :N], torch.full((m, N), 7.0, device=DEV))
        assert torch.equal(C_.double(), A.double() @ B[:, :N].double()), N


@pytest.mark.parametrize("m,k,rows", [(600, 700, [0, 1, 2, 3, 4, 5, 6, 7]), (2000, 1800, list(range(0, 2000, 97))), (16384, 600, [5, 6000, 16383]), (1000, 4096, [999])])
def test_long_rows_of_a_dense_matrix_in_turns(m, k, rows):
    """Long rows beside each other and far apart, in places that the XCDs of a shared tile take in turns: one to seven tiles of 64 columns, whole eights and more."""
    print(f"dense, long rows in turns: {m}x{k}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(m)
    share = torch.full((m, 1), 0.001, device=DEV)
    share[torch.tensor(rows)] = 0.95
    A = torch.randint(1, 8, (m, k), generator=g, device=DEV, dtype=torch.float32) * (torch.rand((m, k), generator=g, device=DEV) < share)
    B = torch.randint(-8, 9, (k, 700), generator=g, device=DEV, dtype=torch.float32)
    H = binding.gcoo_from_dense(A, 32)
    for N in (4, 16, 33, 64, 100, 150, 200, 300, 420, 512, 700):
        C_ = binding.gcoo_spdm(H, B[:, :N], torch.full((m, N), 7.0, device=DEV))
        assert torch.equal(C_.double(), A.double() @ B[:, :N].double()), N
