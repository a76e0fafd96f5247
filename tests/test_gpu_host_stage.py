"""A host CSR input waits in pinned buffers of the library: more conversions in flight than there are buffers, from one thread and from
several, inputs that do not fit one, groups of more than 64 rows (one copy to the device instead), and the caller's arrays overwritten as
soon as the call returns.  Against the CPU oracle."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding, workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _convert_many(ws, p, handles):
    for w in ws:
        arrays = [w.row_ptr.copy(), w.col_idx.copy(), w.vals.copy()]
        handles.append((w, binding.gcoo_from_csr(w.m, w.k, *arrays, p, device=DEV)))
        for x in arrays:
            x.fill(1)                                          # the call has what it needs


def _check(handles, p):
    for w, A in handles:
        want, e = orc.gcoo_from_csr(w.m, w.k, w.row_ptr, w.col_idx, w.vals, p), A.export()
        for key in ("rows", "cols", "gIdxes", "nnzPerGroup"):
            assert np.array_equal(e[key], getattr(want, key)), key
        assert np.array_equal(e["values"].view(np.uint32), want.values.view(np.uint32))


@pytest.mark.parametrize("p,m,k", [(32, 500, 700), (128, 300, 400), (32, 40, 60000)])
def test_more_in_flight_than_buffers(p, m, k):
    print(f"host stage: p={p} {m}x{k}", flush=True)
    handles = []
    _convert_many([workloads.uniform_random(m, k, 1, 0.97, seed=i) for i in range(9)], p, handles)
    _check(handles, p)


def test_an_input_that_does_not_fit():
    print("host stage: 600000 entries", flush=True)
    handles = []
    _convert_many([workloads.uniform_random(3000, 2000, 1, 0.9, seed=5)], 32, handles)
    _check(handles, 32)


def test_from_several_threads():
    print("host stage: six threads", flush=True)
    sets = [[workloads.uniform_random(200 + 10 * t, 300, 1, 0.9, seed=10 * t + i) for i in range(4)] for t in range(6)]
    outs = [[] for _ in sets]
    threads = [threading.Thread(target=_convert_many, args=(ws, 32, out)) for ws, out in zip(sets, outs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for ws, out in zip(sets, outs):
        assert len(out) == len(ws)
        _check(out, 32)


@pytest.mark.parametrize("m,k,p,lens", [
    (512, 300, 1, 3), (513, 300, 1, 3),                       # as many groups as the launch says the starts of, and one more
    (70, 4096, 32, 40), (70, 4097, 32, 40),                   # the last column that one launch takes (1024 threads), and one more
    (130, 900, 50, 9), (64, 1, 64, 1),                        # masks of two words; one column
    (40, 500, 32, [0] * 20 + [500] * 6 + [0] * 14),           # more entries in a group than its threads take at once; empty rows and a nearly empty group
    (96, 2500, 32, [0] * 32 + [33] * 32 + [0] * 32),          # groups without an entry
])
def test_one_launch_from_host_memory(m, k, p, lens):
    print(f"host stage, one launch: {m}x{k} p={p}", flush=True)
    rng = np.random.default_rng(m + k)
    lens = np.full(m, lens) if np.isscalar(lens) else np.array(lens)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([rng.permutation(np.r_[k - 1, rng.choice(k - 1, n - 1, replace=False)] if n > 1 else [k - 1] * n) for n in lens]).astype(np.int32)
    w = workloads.Workload("host", m, k, 70, rp, ci, rng.standard_normal(len(ci)).astype(np.float32), rng.standard_normal((k, 70)).astype(np.float32))
    for twice in (False, True):
        if twice and lens[33 % m] > 1:                         # a coordinate repeated
            w.col_idx[rp[33 % m]] = w.col_idx[rp[33 % m] + 1]
        handles = []
        _convert_many([w], p, handles)
        _check(handles, p)
        C = binding.gcoo_spdm(handles[0][1], torch.from_numpy(w.B).to(DEV))
        C64, D64 = orc.spdm_csr(w.k, w.N, w.row_ptr, w.col_idx, w.vals, w.B)
        err, bad = orc.max_scaled_error(C.cpu().numpy(), C64, D64)
        assert bad == 0 and err < 2e-6, (err, bad)


@pytest.mark.parametrize("m,k", [(3000, 4000), (33, 65536), (33, 65537)])
def test_two_launches_from_host_memory(m, k):
    """Columns of 16 bits as far as they go, and of 32 bits beyond."""
    print(f"host stage, two launches: {m}x{k}", flush=True)
    w = workloads.uniform_random(m, k, 1, 1 - 100000 / (m * k), seed=m)
    w.col_idx[w.row_ptr[1] - 1] = k - 1                        # (the last column, in order)
    handles = []
    _convert_many([w], 32, handles)
    _check(handles, 32)
