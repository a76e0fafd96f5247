"""The row-by-row kernel (the automatic choice for short rows and for small and narrow products) at the sizes where it can go
wrong: batches of 16 entries full and one over, rows shared by a wave and by a workgroup, every width of a slot, tiles that
begin inside a 128-byte line, entries of a dense input brought back into row order.  Against the CPU oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding, workloads
from tests.host_calls import SUMS

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _rows_of_lengths(lens, k, N, seed):
    """CSR with the given row lengths (columns distinct while they fit, repeated beyond), B dense."""
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(k, n, replace=n > k)).astype(np.int32) for n in lens]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate(cols) if len(lens) else np.zeros(0, np.int32)
    va = rng.standard_normal(len(ci)).astype(np.float32)
    return workloads.Workload("lens", len(lens), k, N, rp, ci, va, rng.standard_normal((k, N)).astype(np.float32))


def _check(w, p, shift=0, pad=0, dense=False):
    Bbig = torch.zeros((w.k, w.N + shift + pad), device=DEV)
    Bbig[:, shift:shift + w.N] = torch.from_numpy(w.B).to(DEV)
    Cbig = torch.full((w.m, w.N + shift + pad + 8), 7.0, device=DEV)
    Bv, Cv = Bbig[:, shift:shift + w.N], Cbig[:, shift:shift + w.N]
    dev = [torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)]
    if dense:
        Ah = np.zeros((w.m, w.k), np.float32)
        Ah[np.repeat(np.arange(w.m), np.diff(w.row_ptr)), w.col_idx] = w.vals
        A = binding.gcoo_from_dense(torch.from_numpy(Ah).to(DEV), p)
    else:
        A = binding.gcoo_from_csr(w.m, w.k, *dev, p, known_nnz=True)
    binding.gcoo_spdm(A, Bv, Cv)
    torch.cuda.synchronize()
    C64, D64 = orc.spdm_csr(w.k, w.N, w.row_ptr, w.col_idx, w.vals, w.B)
    err, bad = orc.max_scaled_error(Cv.cpu().numpy(), C64, D64)
    assert bad == 0 and err < 2e-6, (err, bad)
    assert torch.all(Cbig[:, :shift] == 7.0) and torch.all(Cbig[:, shift + w.N:] == 7.0)
    first = Cv.clone()
    binding.gcoo_spdm(A, Bv, Cv)
    assert torch.equal(first, Cv)                          # the same bits on every run


@pytest.mark.parametrize("N,shift,pad", [(4, 0, 0), (5, 0, 0), (16, 0, 0), (17, 1, 2), (32, 0, 0), (33, 0, 0), (64, 0, 0), (65, 3, 0), (128, 0, 0),
                                         (131, 2, 3), (260, 0, 0), (1031, 1, 0)])
def test_widths_and_alignments(N, shift, pad):
    print(f"rows: N={N} shift={shift} pad={pad}", flush=True)
    _check(_rows_of_lengths([0, 1, 15, 16, 17, 31, 32, 33, 2, 0, 7, 48, 64, 65, 3, 5, 90] * 3, 211, N, seed=N), 32, shift, pad)


@pytest.mark.parametrize("p,dense", [(8, False), (32, True), (64, False), (64, True), (128, True)])
def test_long_rows_shared_by_a_wave_and_by_a_workgroup(p, dense):
    """Rows just below and above the lengths from which a wave and a workgroup take them, several in one workgroup."""
    rng = np.random.default_rng(p)
    lens = np.minimum(rng.zipf(1.6, 400), 40)
    lens[[3, 4, 5, 40, 41, 200]] = [65, 64, 512, 513, 1900, 2000]
    lens[-1] = 700
    print(f"rows: long rows p={p} dense={dense}", flush=True)
    _check(_rows_of_lengths(lens, 2048, 68, seed=p), p, dense=dense)


@pytest.mark.parametrize("m,k,N,n", [(1, 1, 4, 1), (1, 5000, 64, 120), (3, 300, 260, 100), (64, 300, 64, 100), (5000, 9, 40, 2), (40000, 3000, 20, 3)])
def test_few_and_many_rows(m, k, N, n):
    print(f"rows: m={m} k={k} N={N}, {n} entries each", flush=True)
    _check(_rows_of_lengths([n] * m, k, N, seed=m), 32)


@pytest.mark.parametrize("N", [1, 2, 3])
def test_one_two_and_three_columns(N):
    print(f"rows: N={N}", flush=True)
    _check(_rows_of_lengths([0, 1, 15, 16, 17, 100, 3] * 7, 300, N, seed=N), 32, shift=1, pad=1)


def test_b_of_more_than_4_gb():
    """Offsets of rows of B beyond 32 bits."""
    w = _rows_of_lengths([0, 20, 40, 3, 70] * 9, 2100, 72, seed=6)
    print("rows: B of 8.8 GB", flush=True)
    _check(w, 32, pad=(1 << 20) - 72)


def test_repeated_and_non_finite():
    """Repeated coordinates add up; a row of B that no entry touches may hold anything."""
    w = _rows_of_lengths([30, 0, 5, 17] * 20, 12, 36, seed=4)              # more entries than columns: coordinates repeat
    _check(w, 16)
    w = _rows_of_lengths([3, 9, 0, 20] * 10, 400, 36, seed=5)
    w.B[np.setdiff1d(np.arange(w.k), w.col_idx)] = np.inf
    _check(w, 16)


@pytest.mark.parametrize("k,N,times", [(7000, 131, 9), (9001, 1501, 9), (6600, 3401, 375), (3000, 2504, 500)])
def test_a_few_entries_per_row_of_many_columns(k, N, times):
    """Rows short enough for the wide tiles whatever k is, and one row beyond: 16 entries and more beside them; the last two with a whole
    wave per row."""
    print(f"rows: few entries, k={k} N={N}", flush=True)
    lens = [0, 3, 9, 1, 7, 12, 2, 16, 5, 17, 4, 6, 8, 0, 1, 40] if times < 10 else [0, 3, 9, 1, 1, 0, 2, 0, 5, 17, 4, 0, 0, 0, 1, 20]
    _check(_rows_of_lengths(lens * times, k, N, seed=k), 32)


@pytest.mark.parametrize("p", [32, 100])
def test_row_pitch_of_b_beyond_32_bits(p):
    """Rows of B 2^30 elements apart and one element more, which the automatic choice leaves to the LDS kernel, and one element less."""
    w = _rows_of_lengths([0, 2, 1, 3] * 9, 3, 68, seed=8)
    dev = [torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)]
    A = binding.gcoo_from_csr(w.m, w.k, *dev, p, known_nnz=True)
    C64, D64 = orc.spdm_csr(w.k, w.N, w.row_ptr, w.col_idx, w.vals, w.B)
    room = torch.empty(2 * ((1 << 30) + 1) + w.N, device=DEV)
    for ldb in ((1 << 30) - 1, 1 << 30, (1 << 30) + 1):
        print(f"rows: ldb={ldb} p={p}", flush=True)
        B = room.as_strided((w.k, w.N), (ldb, 1))
        B.copy_(torch.from_numpy(w.B))
        C = binding.gcoo_spdm(A, B)
        err, bad = orc.max_scaled_error(C.cpu().numpy(), C64, D64)
        assert bad == 0 and err < 2e-6, (ldb, err, bad)


@pytest.mark.parametrize("policy", [binding.SHARE_ALWAYS, binding.SHARE_NEVER])
def test_few_columns_of_a_matrix_with_a_run_schedule(policy):
    """More rows and entries than the automatic choice takes row by row where the matrix has a run schedule, whose kernel has no
    instance for so few columns."""
    rng = np.random.default_rng(policy)
    m, k, n = 33000, 900, 30
    rp = (np.arange(m + 1) * n).astype(np.int32)
    ci = np.sort(rng.integers(0, k, (m, n)), axis=1).astype(np.int32).reshape(-1)
    va = rng.standard_normal(m * n).astype(np.float32)
    binding.gcoo_set_share_policy(policy)
    try:
        A = binding.gcoo_from_csr(m, k, *[torch.from_numpy(x).to(DEV) for x in (rp, ci, va)], 32, known_nnz=True)
    finally:
        binding.gcoo_set_share_policy(binding.SHARE_AUTO)
    for N in (1, 2, 3, 4):
        print(f"rows: run schedule, policy={policy} N={N}", flush=True)
        B = rng.standard_normal((k, N)).astype(np.float32)
        C = binding.gcoo_spdm(A, torch.from_numpy(B).to(DEV))
        C64, D64 = orc.spdm_csr(k, N, rp, ci, va, B)
        err, bad = orc.max_scaled_error(C.cpu().numpy(), C64, D64)
        assert bad == 0 and err < 2e-6, (N, err, bad)


@pytest.mark.parametrize("p,policy", [(1, binding.SHARE_AUTO), (32, binding.SHARE_AUTO), (32, binding.SHARE_NEVER), (128, binding.SHARE_AUTO)])
def test_no_columns(p, policy):
    """A of k = 0 columns: zeros, in all N columns of C and nowhere else."""
    binding.gcoo_set_share_policy(policy)
    try:
        A = binding.gcoo_from_csr(70, 0, np.zeros(71, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32), p, device=DEV)
    finally:
        binding.gcoo_set_share_policy(binding.SHARE_AUTO)
    for N in (1, 3, 4, 130):
        for variant in (binding.VARIANT_AUTO, binding.VARIANT_REG) if N >= 4 else (binding.VARIANT_AUTO,):
            print(f"rows: no columns, p={p} N={N} variant={variant}", flush=True)
            C = torch.full((70, N + 5), 7.0, device=DEV)
            binding.gcoo_spdm(A, torch.empty((0, N), device=DEV), C[:, :N], variant=variant)
            assert not C[:, :N].any() and torch.all(C[:, N:] == 7.0)


@pytest.mark.parametrize("m,k,N,lens,shift,pad", [(300, 211, 203, [0, 1, 2, 3, 9], 1, 0), (300, 211, 995, [0, 1, 2, 3, 9], 2, 1), (13500, 300, 1501, [0, 1, 2, 3, 5], 3, 0),
                                                  (90, 200, 1103, [60, 1, 17], 1, 2), (150, 6600, 77, [40, 0, 33], 2, 0), (150, 6600, 129, [40, 0, 33], 0, 0),
                                                  (130, 9100, 1030, [7, 9, 0], 1, 0), (130, 9100, 1030, [70, 9, 0], 1, 0), (1003, 2700, 129, [60, 53, 70], 1, 0), (1003, 2700, 208, [60, 53, 70], 0, 1),
                                                  (1003, 2700, 129, [40, 0, 33], 1, 0), (1003, 2700, 160, [40, 0, 33], 2, 1), (1003, 2700, 897, [40, 7], 1, 0),
                                                  (9001, 11000, 135, [5, 0, 7], 1, 0), (2100, 2700, 317, [5, 0, 7], 1, 0), (1040, 2700, 1047, [5, 0, 7], 0, 0),
                                                  (130, 8100, 1030, [7, 4, 0], 1, 0), (130, 9100, 7300, [9, 4, 0], 1, 0)])
def test_widths_of_tiles_and_tiles_moved_to_whole_lines(m, k, N, lens, shift, pad):
    """64, 128 and 256 columns per tile, moved down to whole lines of C (rows of a few entries) and not."""
    print(f"rows: tiles m={m} k={k} N={N} lens={lens} shift={shift}", flush=True)
    _check(_rows_of_lengths(np.resize(lens, m), k, N, seed=m + N), 32, shift, pad)


@pytest.mark.parametrize("N", [64, 131, 323, 452, 515, 580])
def test_long_rows_in_turns_over_the_xcds_of_a_tile(N):
    """1 to 10 tiles of 64 columns, those beyond the last eight cut into slices that begin and end inside a tile; long rows at both ends of the matrix and between."""
    print(f"rows: long rows in turns N={N}", flush=True)
    lens = np.full(3001, 150)
    lens[:90] = lens[2950:] = lens[500:2500:9] = 1300
    _check(_rows_of_lengths(lens, 12000, N, seed=N), 32, 1 if N % 2 else 0)


@pytest.mark.parametrize("m,k,N,lens", [(17000, 900, 16, [3, 0, 9]), (7001, 900, 16, [30, 2]), (7001, 900, 29, [3, 0, 40]), (900, 7000, 31, [130, 250]), (50, 7000, 63, [900, 130, 121]), (601, 5000, 200, [300, 0, 140])])
def test_narrow_tiles_and_rows_of_many_entries(m, k, N, lens):
    """Four, eight and sixteen lanes to a row; rows of so many entries that all slots of a wave take one at a time."""
    print(f"rows: narrow m={m} k={k} N={N} lens={lens}", flush=True)
    _check(_rows_of_lengths(np.resize(lens, m), k, N, seed=m + N), 32, 1 if N % 2 else 0)


@pytest.mark.parametrize("lens", [[1536, 1537], [1537, 1537, 1537], [513, 1536], [512, 600, 2500, 0]])
@pytest.mark.parametrize("dense", [False, True])
def test_longest_rows_from_the_front_of_the_list(lens, dense):
    """Rows just below and above the lengths from which a row is listed, and from the front: one class alone and both, the list filled from both sides."""
    print(f"rows: longest first lens={lens} dense={dense}", flush=True)
    _check(_rows_of_lengths(np.resize(lens + [3] * 20, 301), 9000, 67, seed=len(lens)), 32, dense=dense)


def _added_up(terms, sums, eights):
    """The sum over the entries (axis 1) in the order that a slot with a row to itself has: in one chain; in `sums` chains of every sums-th entry; eight by themselves first."""
    if eights:
        total = np.zeros_like(terms[:, 0])
        for at in range(0, terms.shape[1], 8):
            part = terms[:, at].copy()
            for i in range(at + 1, min(at + 8, terms.shape[1])):
                part += terms[:, i]
            total += part
        return total
    chains = []
    for s in range(sums):
        chains.append(np.zeros_like(terms[:, 0]))
        for i in range(s, terms.shape[1], sums):
            chains[s] += terms[:, i]
    return chains[0] if sums == 1 else chains[0] + chains[1]


@pytest.mark.parametrize("lanes,ahead,sums,m,k,N,per_row", SUMS)
def test_a_row_that_narrower_slots_would_share_is_no_less_exact(lanes, ahead, sums, m, k, N, per_row):
    """Every product is exact, so the bits of a sum show the order of it.  (Which instance serves a shape: tests/test_host_calls.py.)"""
    print(f"rows: {sums} sums, {lanes} lanes, N={N}", flush=True)
    rng = np.random.default_rng(N)
    w = _rows_of_lengths([per_row] * m, k, N, seed=N)
    w.B[:] = 2.0 ** rng.integers(-3, 4, (k, N)) * rng.choice([-1.0, 1.0], (k, N))
    A = binding.gcoo_from_csr(m, k, *[torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)], 32, known_nnz=True)
    C = binding.gcoo_spdm(A, torch.from_numpy(w.B).to(DEV)).cpu().numpy()
    terms = w.vals.reshape(m, per_row, 1) * w.B[w.col_idx.reshape(m, per_row)]
    assert np.array_equal(C, _added_up(terms, sums, eights=sums > 1 and (lanes == 64 or ahead == 8)))
    if sums > 1 and per_row > 16:
        exact = terms.sum(1, dtype=np.float64)
        assert np.linalg.norm(C - exact) < 0.85 * np.linalg.norm(_added_up(terms, 1, False) - exact)
