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
