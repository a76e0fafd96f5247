"""The register kernel (spdm_sched, spdm_sched_coop), which reads the run schedule that conversions build under GCOO_SHARE_NEVER and
GCOO_SHARE_ALWAYS: any N and alignment in each of its layouts, heavy groups split over a workgroup, launches of few items, full size.
Every test makes sure that this is the kernel that runs.  Against the CPU oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding, workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def run_schedule():
    binding.gcoo_set_share_policy(binding.SHARE_NEVER)
    yield
    binding.gcoo_set_share_policy(binding.SHARE_AUTO)


def _check(w, A, shift=0, pad=0, r0=0, r1=None):
    """C = A x B through GCOO_VARIANT_REG twice, with guard columns around C: rows [r0, r1) against the oracle, the same bits."""
    r1 = w.m if r1 is None else r1
    Bv = torch.zeros((w.k, w.N + shift + pad), device=DEV)[:, shift:shift + w.N]
    Bv.copy_(torch.from_numpy(w.B))
    C64, D64 = orc.spdm_csr(w.k, w.N, w.row_ptr, w.col_idx, w.vals, w.B, r0, r1)
    outs = []
    for _ in range(2):
        Cbig = torch.full((w.m, w.N + shift + pad), 7.0, device=DEV)
        Cv = Cbig[:, shift:shift + w.N]
        assert binding.gcoo_spdm_kernel(A, Bv, Cv, binding.VARIANT_REG) == binding.KERNEL_SCHED
        binding.gcoo_spdm(A, Bv, Cv, variant=binding.VARIANT_REG)
        assert torch.all(Cbig[:, :shift] == 7.0) and torch.all(Cbig[:, shift + w.N:] == 7.0)
        outs.append(Cv)
    assert torch.equal(*outs)
    err, bad = orc.max_scaled_error(outs[0][r0:r1].cpu().numpy(), C64, D64)
    assert bad == 0 and err < 2e-6, (err, bad)


def _convert(w, p):
    return binding.gcoo_from_csr(w.m, w.k, *[torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)], p, known_nnz=True)


@pytest.mark.parametrize("p", [1, 8, 32, 38, 48, 64, 100])
@pytest.mark.parametrize("N,shift,pad", [(4, 0, 0), (7, 1, 2), (256, 0, 0), (1031, 0, 0), (1029, 1, 11), (1024, 2, 14)])
def test_widths_and_alignments(p, N, shift, pad):
    w = workloads.uniform_random(300, 400, N, 0.9, seed=31)
    print(f"run schedule: p={p} N={N} shift={shift} pad={pad}", flush=True)
    _check(w, _convert(w, p), shift, pad)


@pytest.mark.parametrize("m,k,N,p,sparsity", [(64, 6000, 256, 32, 0.5), (40, 3000, 520, 16, 0.7), (128, 5000, 128, 64, 0.8), (33, 9000, 64, 32, 0.97),
                                              (256, 2500, 1024, 32, 0.9)])
def test_heavy_groups(m, k, N, p, sparsity):
    """Few (group, tile) items with thousands of entries each: eight waves share a group and add up their sums in a fixed order."""
    w = workloads.uniform_random(m, k, N, sparsity, seed=m + k + N)
    print(f"run schedule: heavy groups m={m} k={k} N={N} p={p}", flush=True)
    _check(w, _convert(w, p))


@pytest.mark.parametrize("p", [4, 16, 32, 38, 64])
@pytest.mark.parametrize("N", [64, 260, 1031])
def test_skewed_rows_in_launches_of_few_items(p, N):
    w = workloads.zipf_rows(900, 5000, N, seed=23 + p, row_max=3000)
    print(f"run schedule: skewed rows p={p} N={N} nnz={w.nnz}", flush=True)
    _check(w, _convert(w, p))


def test_dense_input_and_unsorted_rows():
    w = workloads.uniform_random(500, 700, 132, 0.93, seed=6)
    Ah = np.zeros((w.m, w.k), np.float32)
    Ah[np.repeat(np.arange(w.m), np.diff(w.row_ptr)), w.col_idx] = w.vals
    print("run schedule: dense input, unsorted rows", flush=True)
    _check(w, binding.gcoo_from_dense(torch.from_numpy(Ah).to(DEV), 32))
    rng = np.random.default_rng(2)
    for b, e in zip(w.row_ptr[:-1], w.row_ptr[1:]):
        perm = rng.permutation(e - b)
        w.col_idx[b:e], w.vals[b:e] = w.col_idx[b:e][perm], w.vals[b:e][perm]
    _check(w, _convert(w, 32))


@pytest.mark.parametrize("index,p", [(1, 32), (2, 38), (3, 32), (4, 32)])
def test_named_workloads(index, p):
    w = workloads.config(index)
    print(f"run schedule: config{index} p={p} nnz={w.nnz}", flush=True)
    r1 = w.m if w.nnz * w.N < 3e9 else 1600
    _check(w, _convert(w, p), r1=r1)
