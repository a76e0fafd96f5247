"""The sixteen-wave kernel that reads the band schedule, at the sizes where it can go wrong: one, two and three bands full and with
one column over, lists with one unit and with several, last steps of a unit, more rows than a block, widths around a tile,
rows of B aligned to 4 bytes only, repeated coordinates.  Against the CPU oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding, workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _run(w, p, variant, shift=0, pad=0, kernel=None):
    Bbig = torch.zeros((w.k, w.N + shift + pad), device=DEV)
    Bbig[:, shift:shift + w.N] = torch.from_numpy(w.B).to(DEV)
    dev = [torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)]
    outs = []
    for _ in range(2):                                     # two conversions: the same bits
        A = binding.gcoo_from_csr(w.m, w.k, *dev, p, known_nnz=True)
        Cbig = torch.full((w.m, w.N + shift + pad + 8), 7.0, device=DEV)
        Cv = Cbig[:, shift:shift + w.N]
        assert kernel is None or binding.gcoo_spdm_kernel(A, Bbig[:, shift:shift + w.N], Cv, variant) == kernel
        binding.gcoo_spdm(A, Bbig[:, shift:shift + w.N], Cv, variant=variant)
        torch.cuda.synchronize()
        assert torch.all(Cbig[:, :shift] == 7.0) and torch.all(Cbig[:, shift + w.N:] == 7.0)
        outs.append(Cv.clone())
    assert torch.equal(outs[0], outs[1])
    C64, D64 = orc.spdm_csr(w.k, w.N, w.row_ptr, w.col_idx, w.vals, w.B)
    err, bad = orc.max_scaled_error(outs[0].cpu().numpy(), C64, D64)
    assert bad == 0 and err < 2e-6, (err, bad)


def _columns_used(m, k, used, per_row, N, seed):
    """m rows of `per_row` entries in `used` of k columns (all of them used)."""
    rng = np.random.default_rng(seed)
    cols = np.sort(rng.choice(k, used, replace=False))
    pick = np.stack([np.sort(rng.choice(used, per_row, replace=False)) for _ in range(m)])
    for u in range(used):                                  # every column at least once
        if not (pick == u).any():
            pick[u % m, 0] = u
            pick[u % m].sort()
    rp = (np.arange(m + 1) * per_row).astype(np.int32)
    return workloads.Workload("used", m, k, N, rp, cols[pick].reshape(-1).astype(np.int32),
                              rng.standard_normal(m * per_row).astype(np.float32), rng.standard_normal((k, N)).astype(np.float32))


@pytest.mark.parametrize("m,used,per_row,N", [(1, 60, 60, 4), (40, 80, 70, 256), (384, 81, 60, 260), (300, 160, 64, 512), (400, 161, 64, 252), (777, 240, 62, 516),
                                              (97, 241, 130, 64)])
def test_bands_full_and_one_column_over(m, used, per_row, N):
    """3500 columns, of which few are used, at 1.5 % density and more: the shapes for which GCOO_VARIANT_SHARE is served."""
    print(f"band: m={m} used={used} per_row={per_row} N={N}", flush=True)
    _run(_columns_used(m, 3500, used, per_row, N, seed=m + used), 32, binding.VARIANT_SHARE)


@pytest.mark.parametrize("m,used,per_row,N", [(384, 150, 150, 260), (384, 160, 150, 256), (385, 161, 150, 4), (400, 240, 150, 512), (777, 241, 150, 252), (384, 319, 60, 260),
                                              (768, 320, 60, 128), (769, 321, 60, 4), (777, 480, 62, 252), (97, 481, 130, 64), (385, 160, 60, 132)])
def test_bands_of_both_cuts(m, used, per_row, N):
    """150 entries per row: the wide cut (bands of 80 rows of B, 24 rows of A per wave at most); 60 and 130: the tall one (160 and 48)."""
    print(f"band, both cuts: m={m} used={used} per_row={per_row} N={N}", flush=True)
    _run(_columns_used(m, 3500, used, per_row, N, seed=m + used), 32, binding.VARIANT_SHARE, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("m,used,per_row,N", [(2600, 150, 150, 260), (2600, 160, 150, 256), (4601, 161, 150, 4), (4600, 240, 150, 512), (4607, 241, 150, 252), (4608, 319, 60, 260),
                                              (4608, 320, 60, 128), (4609, 321, 60, 4), (4700, 480, 62, 252), (2700, 160, 60, 132), (1500, 320, 150, 64), (1000, 240, 205, 64)])
def test_bands_of_both_cuts_with_many_and_few_rows_per_wave(m, used, per_row, N):
    """Matrices of so many rows that the blocks fill the compute units with 12 to 48 rows per wave, and of fewer."""
    print(f"band, both cuts: m={m} used={used} per_row={per_row} N={N}", flush=True)
    _run(_columns_used(m, 3500, used, per_row, N, seed=m + used), 32, binding.VARIANT_SHARE, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("m,k,N,per_row", [(301, 2962, 2427, 350), (300, 4511, 4504, 300), (120, 6000, 6000, 900), (1836, 2885, 1836, 577)])
def test_few_rows_per_wave(m, k, N, per_row):
    """Fewer than twelve, in both cuts."""
    print(f"band, few rows: m={m} k={k} N={N} per_row={per_row}", flush=True)
    _run(workloads.uniform_random(m, k, N, 1 - per_row / k, seed=m + N), 32, binding.VARIANT_AUTO, 1, 1, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("m,k,N,s,shift,pad", [(4000, 4000, 2044, 0.98, 0, 0), (5000, 5001, 2501, 0.995, 0, 0), (5000, 5001, 2500, 0.995, 1, 0)])
def test_automatic_choice_of_both_cuts(m, k, N, s, shift, pad):
    """The wide cut with few entries per band; the tall one with rows of B aligned to 4 bytes only, its last tile inside the one before."""
    print(f"band, both cuts, automatic: m={m} k={k} N={N} s={s} shift={shift}", flush=True)
    _run(workloads.uniform_random(m, k, N, s, seed=m + N), 32, binding.VARIANT_AUTO, shift, pad, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("m,k,N,nnz", [(4000, 4000, 2045, 320000), (5600, 5601, 2601, 90000), (1000, 3000, 2045, 150000), (4000, 4000, 2045, 224000)])
@pytest.mark.parametrize("shift,pad", [(1, 0), (2, 1), (3, 2)])
def test_requests_spread_over_a_band_from_rows_aligned_to_4_bytes(m, k, N, nnz, shift, pad):
    """Sixteen bytes per lane from any multiple of four bytes straight to LDS: by the late half behind its first unit, a row at a time and step in the tall cut and in the wide one, and by the late half behind its second
    step."""
    print(f"band, spread requests: m={m} k={k} N={N} shift={shift} pad={pad}", flush=True)
    _run(workloads.uniform_random(m, k, N, 1 - nnz / (m * k), seed=m + N), 32, binding.VARIANT_AUTO, shift, pad, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("m,k,per_row,N", [(4000, 4000, 40, 2605), (5000, 5001, 47, 2605), (5000, 5001, 42, 2605), (4000, 4000, 160, 2053), (4000, 4000, 120, 2053), (4000, 4000, 76, 2053)])
@pytest.mark.parametrize("even", [True, False])
def test_requests_of_the_late_half_behind_the_first_and_the_second_unit(m, k, per_row, N, even):
    """Both cuts, on both sides of the number of entries from which the late half asks behind its second unit, by its first one below; waves of one unit to a band beside waves of many."""
    print(f"band, late half: m={m} k={k} per_row={per_row} even={even}", flush=True)
    rng = np.random.default_rng(m + per_row)
    n = np.full(m, per_row) if even else np.resize(np.repeat([per_row // 8, 2 * per_row, per_row // 2, 3 * per_row // 2], 40), m)
    rp = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(k, x, replace=False)) for x in n]).astype(np.int32)
    _run(workloads.Workload("late", m, k, N, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), rng.standard_normal((k, N)).astype(np.float32)),
         32, binding.VARIANT_AUTO, kernel=binding.KERNEL_BAND)


def test_tall_cut_with_repeated_coordinates_and_infinities():
    """Lists that are written the slow way, of more than 32 rows; rows of B that no entry touches hold infinities."""
    rng = np.random.default_rng(21)
    m, k, N = 900, 3500, 132
    rows = [np.concatenate([rng.choice(3400, 58, replace=False), [17] * (i % 5), [3000] * (i % 3)]).astype(np.int32) for i in range(m)]
    for x in rows:
        rng.shuffle(x)
    rp = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.int32)
    ci = np.concatenate(rows)
    B = rng.standard_normal((k, N)).astype(np.float32)
    B[3400:] = np.inf
    print("band, tall: repeated coordinates", flush=True)
    _run(workloads.Workload("repeated", m, k, N, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), B), 32, binding.VARIANT_SHARE, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("m,k,lens,twice", [(777, 3500, [0, 1, 200, 3, 0, 0, 130, 64, 65, 63], ()), (800, 3500, [150] * 40 + [320] * 16, ()), (900, 3500, [170], ()),
                                            (400, 3500, [0] * 15 + [900], ()), (60, 20000, [700], (19999,)), (60, 20000, [700], (3,)), (130, 30000, [900, 0, 500], (29999,))])
def test_rows_of_all_lengths(m, k, lens, twice):
    """Lists whose 64 neighbouring entries lie in one row and in many, with empty rows between; of more entries than the threads of a workgroup keep beside
    shorter ones; more distinct columns than are counted at a time, a coordinate repeated among the first of them or the last."""
    print(f"band: m={m} k={k} lens={lens[:4]} twice={twice}", flush=True)
    rng = np.random.default_rng(m + k)
    n = np.resize(lens, m)
    rows = [np.sort(rng.permutation(k)[:x]) for x in n]
    for c in twice:
        for i in range(0, m, 7):
            rows[i] = np.sort(np.concatenate([rows[i][:-2], [c, c]])) if n[i] > 2 else rows[i]
    rp = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    _run(workloads.Workload("lengths", m, k, 132, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), rng.standard_normal((k, 132)).astype(np.float32)),
         32, binding.VARIANT_SHARE, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("kind", ["sorted", "unsorted", "twice", "uneven"])
@pytest.mark.parametrize("m,k,per_row,p", [(800, 3500, 150, 32), (800, 3500, 60, 32), (700, 3500, 60, 48), (9000, 9000, 9, 32), (9000, 12000, 12, 40), (3500, 3500, 17, 32),
                                           (400, 13000, 200, 32), (60, 3500, 60, 7)])
def test_groups_and_bands_in_one_launch(m, k, per_row, p, kind):
    """The launch that orders the groups and fills the bands, one and two mask words, columns and places of distinct ones, both cuts, one turn over the columns and more:
    the five arrays bit for bit, and the product by the bands, or row by row where a list is far too long for them, which both parts have to find."""
    print(f"band, with the groups: {m}x{k} {per_row} a row p={p} {kind}", flush=True)
    rng = np.random.default_rng(m + k + p)
    rows = [np.sort(rng.integers(0, k, per_row)) if kind == "twice" and i % 5 == 0 else np.sort(rng.permutation(k)[:per_row]) for i in range(m)]
    if kind == "unsorted":
        rows = [rng.permutation(x) if i % 3 == 0 else x for i, x in enumerate(rows)]
    if kind == "uneven":
        rows[m // 2:m // 2 + 3] = [np.arange(k)] * 3
    rp = np.concatenate([[0], np.cumsum([len(x) for x in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    w = workloads.Workload("both", m, k, 68, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), rng.standard_normal((k, 68)).astype(np.float32))
    e = binding.gcoo_from_csr(m, k, *[torch.from_numpy(x).to(DEV) for x in (rp, ci, w.vals)], p, known_nnz=True).export()
    want = orc.gcoo_from_csr(m, k, rp, ci, w.vals, p)
    for key in ("rows", "cols", "gIdxes", "nnzPerGroup"):
        assert np.array_equal(e[key], getattr(want, key)), key
    assert np.array_equal(e["values"].view(np.uint32), want.values.view(np.uint32))
    _run(w, p, binding.VARIANT_SHARE if per_row >= 60 and k == 3500 and m > 60 else binding.VARIANT_AUTO)


@pytest.mark.parametrize("m,k,N,s", [(100, 3500, 300, 0.94), (385, 3600, 1024, 0.98), (1000, 7000, 768, 0.995), (50, 20000, 260, 0.97)])
def test_uniform_through_the_share_variant(m, k, N, s):
    print(f"band: m={m} k={k} N={N} s={s}", flush=True)
    _run(workloads.uniform_random(m, k, N, s, seed=m + k), 48, binding.VARIANT_SHARE)


@pytest.mark.parametrize("m,k,N,s,shift,pad", [(4000, 4000, 1001, 0.95, 0, 0), (4000, 4000, 1000, 0.95, 1, 2), (3000, 3000, 2999, 0.7, 0, 0), (5000, 2600, 1280, 0.9, 0, 0)])
def test_automatic_choice_ragged_and_dense(m, k, N, s, shift, pad):
    """The automatic choice of a matrix that has a band schedule (for the first two the row-by-row kernel, for the last two this one): N and rows of
    B that are no multiple of four, runs of pairs."""
    print(f"band, automatic: m={m} k={k} N={N} s={s} shift={shift}", flush=True)
    _run(workloads.uniform_random(m, k, N, s, seed=m + N), 32, binding.VARIANT_AUTO, shift, pad)


def test_repeated_coordinates_and_skewed_rows():
    rng = np.random.default_rng(8)
    rows = []
    for i in range(200):
        c = list(rng.choice(3500, 60, replace=False))
        if i % 9 == 0:
            c += [17] * 45 + [18] * 70
        rng.shuffle(c)                                      # columns of a row in any order
        rows.append(np.array(c, np.int32))
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate(rows)
    w = workloads.Workload("repeated", 200, 3500, 132, rp, ci, rng.standard_normal(len(ci)).astype(np.float32),
                           rng.standard_normal((3500, 132)).astype(np.float32))
    print("band: repeated coordinates", flush=True)
    _run(w, 32, binding.VARIANT_SHARE)
    z = workloads.zipf_rows(500, 3600, 256, seed=2, exponent=1.3, row_max=3500)
    assert 0.015 * z.m * z.k < z.nnz < 0.06 * z.m * z.k
    print("band: skewed rows", flush=True)
    _run(z, 40, binding.VARIANT_SHARE)


@pytest.mark.parametrize("dense,p,N,shift", [(False, 32, 1024, 0), (False, 64, 1021, 1), (True, 32, 1024, 0), (False, 32, 260, 0)])
def test_uneven_rows_are_multiplied_one_by_one(dense, p, N, shift):
    """A matrix that gets a band schedule by its size, with one list of rows of far more entries than the others: the launch of the
    sixteen-wave kernel works row by row.  GCOO_VARIANT_SHARE asks for that kernel where it is served; the automatic choice is the row-by-row kernel
    for a B this narrow, and this one for those of test_automatic_choice_of_this_kernel_for_uneven_rows."""
    print(f"band: uneven rows dense={dense} p={p} N={N}", flush=True)
    rng = np.random.default_rng(N + p)
    m, k = 4000, 3600
    lens = rng.integers(40, 90, m)
    lens[1000:1012] = 3000
    cols = [np.sort(rng.choice(k, n, replace=False)).astype(np.int32) for n in lens]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate(cols)
    w = workloads.Workload("uneven", m, k, N, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), rng.standard_normal((k, N)).astype(np.float32))
    if dense:
        Ah = np.zeros((m, k), np.float32)
        Ah[np.repeat(np.arange(m), lens), ci] = w.vals
        A = binding.gcoo_from_dense(torch.from_numpy(Ah).to(DEV), p)
    else:
        A = binding.gcoo_from_csr(m, k, *[torch.from_numpy(x).to(DEV) for x in (rp, ci, w.vals)], p, known_nnz=True)
    Bbig = torch.zeros((k, N + shift), device=DEV)
    Bbig[:, shift:] = torch.from_numpy(w.B).to(DEV)
    C64, D64 = orc.spdm_csr(k, N, rp, ci, w.vals, w.B)
    for variant in (binding.VARIANT_AUTO, binding.VARIANT_SHARE) if p <= 48 and not shift else (binding.VARIANT_AUTO,):
        C = binding.gcoo_spdm(A, Bbig[:, shift:], variant=variant)
        err, bad = orc.max_scaled_error(C.cpu().numpy(), C64, D64)
        assert bad == 0 and err < 2e-6, (variant, err, bad)
        assert torch.equal(C, binding.gcoo_spdm(A, Bbig[:, shift:], variant=variant))


@pytest.mark.parametrize("m,k,N,s,pad", [(300, 7000, 1000, 0.9955, 0), (700, 7003, 516, 0.995, 4), (385, 7000, 260, 0.9955, 0), (2000, 7000, 300, 0.988, 0)])
def test_few_entries_per_band(m, k, N, s, pad):
    """Waves with no entry in a band, with one step, and with more than the three behind which rows of the next band are requested."""
    print(f"band, few entries: m={m} k={k} N={N} s={s} pad={pad}", flush=True)
    _run(workloads.uniform_random(m, k, N, s, seed=m + k), 32, binding.VARIANT_SHARE, 0, pad)


def test_non_finite_values_beside_uneven_rows_of_a_b_of_almost_4_gb():
    """Uneven rows multiplied one by one by the launch of the sixteen-wave kernel, with rows of B as far up as a descriptor reaches: an
    entry past the end of a row must not load the last ones, which hold infinities and are touched by no entry."""
    rng = np.random.default_rng(14)
    m, k, N, ldb = 400, 131071, 64, 8192
    lens = rng.integers(465, 495, m)
    lens[100:112] = 20000
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(k - 3, n, replace=False)) for n in lens]).astype(np.int32)
    va = rng.standard_normal(len(ci)).astype(np.float32)
    B = rng.standard_normal((k, N)).astype(np.float32)
    B[k - 3:] = np.inf
    Bd = torch.zeros((k, ldb), device=DEV)[:, :N]
    Bd.copy_(torch.from_numpy(B))
    A = binding.gcoo_from_csr(m, k, *[torch.from_numpy(x).to(DEV) for x in (rp, ci, va)], 32, known_nnz=True)
    C64, D64 = orc.spdm_csr(k, N, rp, ci, va, B)
    for variant in (binding.VARIANT_SHARE, binding.VARIANT_AUTO):
        print(f"band: uneven rows, B of 4.29 GB, variant={variant}", flush=True)
        err, bad = orc.max_scaled_error(binding.gcoo_spdm(A, Bd, variant=variant).cpu().numpy(), C64, D64)
        assert bad == 0 and err < 2e-6, (variant, err, bad)


@pytest.mark.parametrize("m,k,N,s,shift,pad", [(4000, 3000, 1001, 0.9, 0, 0), (4000, 3000, 1021, 0.9, 1, 1), (4000, 4000, 2052, 0.95, 1, 2),
                                               (4000, 4000, 2044, 0.95, 4, 4), (30000, 3600, 513, 0.95, 2, 1), (30000, 3600, 257, 0.95, 3, 2)])
def test_automatic_choice_of_this_kernel(m, k, N, s, shift, pad):
    """Wide enough that the automatic choice is this kernel: last tiles that begin inside the tile before, rows of B and C aligned to 4 bytes only."""
    print(f"band, automatic: m={m} k={k} N={N} s={s} shift={shift}", flush=True)
    w = workloads.uniform_random(m, k, N, s, seed=m + N)
    _run(w, 32, binding.VARIANT_AUTO, shift, pad, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("p,N,shift", [(32, 2048, 0), (64, 2045, 1), (32, 2560, 4)])
def test_automatic_choice_of_this_kernel_for_uneven_rows(p, N, shift):
    print(f"band, automatic: uneven rows p={p} N={N} shift={shift}", flush=True)
    rng = np.random.default_rng(N + p)
    m, k = 4000, 3600
    lens = rng.integers(40, 90, m)
    lens[1000:1012] = 3000
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(k, n, replace=False)) for n in lens]).astype(np.int32)
    w = workloads.Workload("uneven", m, k, N, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), rng.standard_normal((k, N)).astype(np.float32))
    _run(w, p, binding.VARIANT_AUTO, shift, 3, kernel=binding.KERNEL_BAND)


@pytest.mark.parametrize("m,N,heavy,long,short,shift", [(9000, 576, 2000, 500, 10, 0), (9000, 64, 2000, 500, 10, 4), (40, 64, 2, 3000, 30, 0), (300, 1100, 3, 3400, 60, 0),
                                                        (5000, 516, 12, 3400, 70, 0), (5000, 96, 12, 3400, 70, 4), (2000, 2052, 40, 2000, 55, 4)])
def test_uneven_rows_in_shares_of_equal_entries(m, N, heavy, long, short, shift):
    """More long rows in a share than there are places for their pieces; fewer rows than shares; one tile, whole eights of tiles and tiles cut into shares; empty rows."""
    print(f"band: uneven rows m={m} N={N} heavy={heavy} shift={shift}", flush=True)
    rng = np.random.default_rng(m + N)
    k = 3500
    lens = np.where(np.arange(m) < heavy, long, short)
    lens[heavy + 3::7] = 0
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(k, n, replace=False)) for n in lens]).astype(np.int32)
    w = workloads.Workload("uneven", m, k, N, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), rng.standard_normal((k, N)).astype(np.float32))
    _run(w, 32, binding.VARIANT_SHARE, shift, shift, kernel=binding.KERNEL_BAND)


def _in_pieces(vals, rows_of_b):
    """The sum of a long row in its pieces: eight of four stretches each, a stretch one entry after the other, the stretches of a piece by pairs, the pieces in their order.
    Every product is exact."""
    terms = vals[:, None] * rows_of_b
    each = -(-len(vals) // 32)
    stretches = np.zeros((32, terms.shape[1]), np.float32)
    for i, term in enumerate(terms):
        stretches[i // each] += term
    s = stretches.reshape(8, 4, -1)
    pieces = (s[:, 0] + s[:, 1]) + (s[:, 2] + s[:, 3])
    total = pieces[0].copy()
    for x in pieces[1:]:
        total += x
    return total


@pytest.mark.parametrize("N,shift", [(2048, 0), (2051, 1)])
def test_uneven_rows_of_many_entries_are_multiplied_once(N, shift):
    """A mean of more than 128 entries, and rows that are long, but less than twice the mean: in pieces and nowhere else, so that the bits do not go by which of two waves is the last."""
    print(f"band: uneven rows of many entries N={N}", flush=True)
    rng = np.random.default_rng(N)
    m, k = 4000, 3600
    lens = rng.integers(130, 170, m)
    lens[1000:1012] = 3000
    long = np.arange(5, m, 50)
    lens[long] = np.resize([255, 256, 257, 258, 288, 289, 310], len(long))
    mean = int(lens.sum()) // m
    assert 155 < mean and 310 < 2 * mean
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(k, n, replace=False)) for n in lens]).astype(np.int32)
    B = (2.0 ** rng.integers(-3, 4, (k, N)) * rng.choice([-1.0, 1.0], (k, N))).astype(np.float32)
    w = workloads.Workload("uneven", m, k, N, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), B)
    _run(w, 32, binding.VARIANT_AUTO, shift, 3, kernel=binding.KERNEL_BAND)
    Bd = torch.from_numpy(B).to(DEV)
    A = binding.gcoo_from_csr(m, k, *[torch.from_numpy(x).to(DEV) for x in (rp, ci, w.vals)], 32, known_nnz=True)
    C = binding.gcoo_spdm(A, Bd).cpu().numpy()
    for r in long[lens[long] > 256]:
        assert np.array_equal(C[r], _in_pieces(w.vals[rp[r]:rp[r + 1]], B[ci[rp[r]:rp[r + 1]]])), (r, lens[r])


def test_export_share_of_a_matrix_with_a_band_schedule():
    """There is no share schedule to copy: nothing but empty arrays, no uninitialised ones."""
    print("band: export_share", flush=True)
    w = workloads.uniform_random(385, 3600, 64, 0.98, seed=5)
    A = binding.gcoo_from_csr(w.m, w.k, w.row_ptr, w.col_idx, w.vals, 32, device=DEV)
    assert {key: x.size for key, x in A.export_share().items()} == dict(hdr=0, blocks=0, sbase=0, ucount=0, ucols=0)
    assert binding.gcoo_from_csr(w.m, w.k, w.row_ptr, w.col_idx, w.vals, 49, device=DEV).export_share() is None
