"""The row-by-row product by a tile of B in LDS, at the sizes where it can go wrong: rows and columns at the edges of a workgroup's LDS, widths one off a tile, rows of
every remainder of a batch, of the open bin of lengths, shared by a wave, repeated coordinates, unaligned operands.  Against the CPU oracle.  (That these shapes
do go by the tile: tests/test_host_calls.py.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding, workloads
from tests.host_calls import TILES

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _matrix(m, k, N, nnz, weights, seed):
    """`nnz` entries, the rows by `weights` but for a few of all lengths around a batch; repeated columns where a row has more entries than there are; non-finite
    rows of B that no entry touches."""
    rng = np.random.default_rng(seed)
    few = np.array([0, 1, 3, 4, 5, 8, 9, 15, 16, 17, 31, 33], np.int64)[:max(1, m // 4)]
    lens = np.concatenate([few, rng.multinomial(nnz - few.sum(), weights(rng, m - len(few)))])
    lens = lens[rng.permutation(m)]
    some = np.sort(rng.permutation(k)[:max(1, k - 3)])                        # the columns that entries have
    ci = np.concatenate([some[np.sort(rng.choice(len(some), n, replace=n > len(some)))] for n in lens]).astype(np.int32)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    B = rng.standard_normal((k, N)).astype(np.float32)
    B[np.setdiff1d(np.arange(k), ci)] = np.inf
    return workloads.Workload("tile", m, k, N, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), B)


def _even(rng, n):
    return np.full(n, 1.0 / n)


def _uneven(rng, n):
    w = rng.zipf(1.6, n).astype(float)
    return w / w.sum()


@pytest.mark.parametrize("weights", [_even, _uneven])
@pytest.mark.parametrize("shift,pad", [(0, 0), (1, 3)])
@pytest.mark.parametrize("case", [t[:4] for t in TILES if t[4]])
def test_tile(case, shift, pad, weights):
    m, k, N, nnz = case
    print(f"tile: {case} {weights.__name__} shift={shift} pad={pad}", flush=True)
    w = _matrix(m, k, N, nnz, weights, seed=m + k)
    Bbig = torch.zeros((k, N + shift + pad), device=DEV)
    Bbig[:, shift:shift + N] = torch.from_numpy(w.B).to(DEV)
    Cbig = torch.full((m + 1, N + shift + 5), 7.0, device=DEV)
    Bv, Cv = Bbig[:, shift:shift + N], Cbig[:m, shift:shift + N]
    A = binding.gcoo_from_csr(m, k, *[torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)], 32, known_nnz=True)
    assert binding.gcoo_spdm_kernel(A, Bv, Cv) == binding.KERNEL_ROWS
    binding.gcoo_spdm(A, Bv, Cv)
    C64, D64 = orc.spdm_csr(k, N, w.row_ptr, w.col_idx, w.vals, w.B)
    err, bad = orc.max_scaled_error(Cv.cpu().numpy(), C64, D64)
    # sums of up to `longest` products in 32 bits, one after the other or in sixteen stretches: errors of 2^-24 each that add up like a random walk (three deviations)
    longest = int(np.diff(w.row_ptr).max())
    assert bad == 0 and err < 2.0 ** -24 * (2 + 3 * longest ** 0.5), (err, bad, longest)
    assert torch.all(Cbig[:m, :shift] == 7.0) and torch.all(Cbig[:, shift + N:] == 7.0) and torch.all(Cbig[m] == 7.0)
    first = Cv.clone()
    Cv.fill_(float("nan"))
    binding.gcoo_spdm(A, Bv, Cv)
    assert torch.equal(first, Cv)                          # the same bits on every run
