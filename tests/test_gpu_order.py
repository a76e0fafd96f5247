"""Ordering a CSR input by column masks where it can go wrong: one part and many, a part that is one column short or over, parts of more
entries than are put in order in LDS (of more distinct columns than a window holds), one, two and eight mask words per column, empty rows at either end, rows whose columns do not
ascend, coordinates that occur twice.  Bit for bit against the CPU oracle, and the product that the rows and bands give."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _csr(m, k, density, kind, seed):
    rng = np.random.default_rng(seed)
    lens = rng.binomial(k, density, m)
    lens[: m // 7] = 0
    lens[-(m // 9 + 1):] = 0 if m > 3 else lens[-1]
    if m > 20:
        lens[m // 2] = k                                           # one full row
    cols = []
    for i, n in enumerate(lens):
        c = np.sort(rng.choice(k, n, replace=False))
        if kind != "sorted" and i % 5 == 0:
            c = rng.permutation(c)
        if kind == "twice" and i % 3 == 0 and n > 1:
            c[rng.integers(1, n)] = c[0]
        cols.append(c.astype(np.int32))
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate(cols).astype(np.int32)
    return rp, ci, rng.standard_normal(len(ci)).astype(np.float32)


@pytest.mark.parametrize("kind", ["sorted", "unsorted", "twice"])
@pytest.mark.parametrize("m,k,density,p", [(1, 1, 1.0, 1), (3, 130, 0.5, 32), (500, 127, 0.2, 32), (500, 128, 0.2, 33), (300, 4096, 0.02, 32),
                                           (300, 4097, 0.02, 31), (300, 8193, 0.01, 32), (130, 2049, 0.05, 64), (400, 300, 0.9, 64),
                                           (400, 1000, 0.3, 65), (600, 513, 0.1, 256), (1500, 700, 0.03, 8), (2100, 900, 0.05, 1),
                                           # many columns per entry of a group: by the places of the distinct columns
                                           (300, 4097, 0.003, 31), (300, 70001, 0.0004, 32), (700, 5000, 0.0005, 64), (520, 9000, 0.0006, 256), (900, 66000, 0.00004, 8),
                                           (2000, 40, 0.004, 1), (70, 1025, 0.002, 33), (3000, 3000, 0.001, 65)])
def test_ordered_by_masks(m, k, density, p, kind):
    print(f"order: {m}x{k} d={density} p={p} {kind}", flush=True)
    rp, ci, va = _csr(m, k, density, kind, seed=m + k + p)
    _check(m, k, rp, ci, va, p)


# 1024 threads for groups of more than 2048 entries and, up to 256 groups, of many columns, 256 otherwise; groups that just fit the LDS and just not, of more
# entries than a thread keeps; rows of more than 512 entries, which have places by group: the first and the last row of a group, all of them, none
@pytest.mark.parametrize("kind", ["sorted", "twice"])
@pytest.mark.parametrize("m,k,entries,p,long", [(8192, 300, 30, 32, []), (8193, 300, 30, 32, []), (8193, 300, 75, 32, []), (64, 4096, 70, 32, []), (64, 4096, 72, 32, []),
                                                (96, 2048, 123, 32, []), (96, 2048, 125, 32, []), (96, 2300, 79, 32, []), (96, 2300, 80, 32, []), (96, 2048, 139, 32, []), (96, 2048, 140, 32, []), (320, 700, 5, 32, [*range(32), 96, 159, 319]),
                                                (9000, 700, 3, 32, [*range(32), 96, 159, 8999]), (9000, 600, 8, 33, [0, 32, 33, 65, 66]),
                                                (300, 2000, 20, 64, [63, 64, 127, 299]), (300, 512, 7, 65, [3, 299]), (200, 513, 2, 1, [0, 77, 199])])
def test_in_one_launch(m, k, entries, p, long, kind):
    print(f"order: {m}x{k} {entries} a row p={p} {len(long)} long rows {kind}", flush=True)
    rng = np.random.default_rng(m + k + entries)
    lens = np.full(m, entries)
    lens[long] = k
    cols = [np.sort(rng.permutation(k)[:n]) for n in lens]
    if kind == "twice":
        for i in (*long[:3], m // 2):
            cols[i][-1] = cols[i][0]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate(cols).astype(np.int32)
    _check(m, k, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), p)


# groups of just so many entries that each of 256 (or 1024) threads has four of them, or eight, one fewer and one more; columns that come to four a thread and to one more
@pytest.mark.parametrize("k", [300, 1024, 1025])
@pytest.mark.parametrize("sizes", [[1023, 1024, 1025, 0, 1, 960, 961], [2047, 2048, 2049, 64, 1984, 1985], [4095, 4096, 4097, 3, 4032, 4033]])
def test_as_many_entries_as_the_threads_take_at_a_time(sizes, k):
    print(f"order: groups of {sizes}, {k} columns", flush=True)
    rng = np.random.default_rng(k + sizes[0])
    lens = np.concatenate([np.diff(np.arange(33) * n // 32) for n in sizes])
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.permutation(k)[:n]) for n in lens]).astype(np.int32)
    _check(len(lens), k, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), 32)


def _check(m, k, rp, ci, va, p):
    want = orc.gcoo_from_csr(m, k, rp, ci, va, p)
    dev = [torch.from_numpy(x).to(DEV) for x in (rp, ci, va)]
    A = binding.gcoo_from_csr(m, k, *dev, p, known_nnz=True)
    e = A.export()
    for key in ("rows", "cols", "gIdxes", "nnzPerGroup"):
        assert np.array_equal(e[key], getattr(want, key)), key
    assert np.array_equal(e["values"].view(np.uint32), want.values.view(np.uint32))
    B = np.random.default_rng(p).standard_normal((k, 20)).astype(np.float32)
    C64, D64 = orc.spdm_csr(k, 20, rp, ci, va, B)
    for variant in (binding.VARIANT_AUTO, binding.VARIANT_LDS):
        got = binding.gcoo_spdm(A, torch.from_numpy(B).to(DEV), variant=variant)
        err, bad = orc.max_scaled_error(got.cpu().numpy(), C64, D64)
        assert bad == 0 and err < 2e-6, (variant, err, bad)
