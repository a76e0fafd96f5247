"""The extension module behind the binding's calls: the same bits as by ctypes, and for arguments that it does not serve what the binding does without it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2005_14469_amd import binding, workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


class _Nothing:
    """Serves no call."""

    def __getattr__(self, name):
        return (lambda h: binding.lib().gcoo_free(h)) if name == "free" else (lambda *args: None)


def _results(w, p):
    dev = [torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)]
    B = torch.from_numpy(w.B).to(DEV)
    dense = torch.zeros((w.m, w.k + 3), device=DEV)[:, :w.k]
    dense[torch.repeat_interleave(torch.arange(w.m, device=DEV), torch.diff(dev[0]).long()), dev[1].long()] = dev[2]
    buf = torch.empty(binding.lib().gcoo_static_handle_bytes(w.m, w.k, len(w.vals), p), dtype=torch.uint8, device=DEV)
    C = torch.full((w.m, w.N + 5), 7.0, device=DEV)
    out = []
    for make in (lambda: binding.gcoo_from_csr(w.m, w.k, *dev, p, known_nnz=True), lambda: binding.gcoo_from_csr(w.m, w.k, *dev, p), lambda: binding.gcoo_from_dense(dense, p),
                 lambda: binding.gcoo_from_csr(w.m, w.k, w.row_ptr, w.col_idx, w.vals, p, device="cuda"),
                 lambda: binding.gcoo_from_csr(w.m, w.k, w.row_ptr.astype(np.int64), np.repeat(w.col_idx, 2)[::2], w.vals.astype(np.float64), p, device=DEV),
                 lambda: binding.gcoo_from_csr_device_static(w.m, w.k, *dev, p, out_buf=buf), lambda: binding.gcoo_from_csr_device_static(w.m, w.k, *dev, p)):
        A = make()
        assert A.shape == (w.m, w.k)
        out += [binding.gcoo_spdm(A, B).cpu(), binding.gcoo_spdm(A, B, C[:, 2:2 + w.N]).cpu(), binding.gcoo_spdm(A, B, variant=binding.VARIANT_LDS).cpu()]
        assert torch.all(C[:, :2] == 7.0) and torch.all(C[:, 2 + w.N:] == 7.0)
        out += [torch.from_numpy(x) for x in A.export().values()]
        A.free()
    return out


@pytest.mark.parametrize("m,k,N,density", [(1, 1, 1, 1.0), (70, 1, 9, 1.0), (1, 90, 33, 0.2), (300, 211, 70, 0.05)])
def test_same_bits_with_and_without_the_module(monkeypatch, m, k, N, density):
    print(f"calls: {m} x {k} x {N}", flush=True)
    w = workloads.uniform_random(m, k, N, 1 - density, seed=m + N)
    by_module = _results(w, 32)
    monkeypatch.setattr(binding, "_calls", _Nothing())
    for x, y in zip(by_module, _results(w, 32), strict=True):
        assert torch.equal(x, y)


def _refused(w, dev):
    A = binding.gcoo_from_csr(w.m, w.k, *dev, 32, known_nnz=True)
    B = torch.from_numpy(w.B).to(DEV)
    freed = binding.gcoo_from_csr(w.m, w.k, *dev, 32, known_nnz=True)
    freed.free()
    bad = w.col_idx.copy()
    bad[0] = w.k
    calls = [lambda: binding.gcoo_spdm(A, B.cpu()), lambda: binding.gcoo_spdm(A, B.double()), lambda: binding.gcoo_spdm(A, B[:-1]), lambda: binding.gcoo_spdm(A, B.t().contiguous().t()),
             lambda: binding.gcoo_spdm(A, B, B), lambda: binding.gcoo_spdm(freed, B), lambda: binding.gcoo_spdm(A, B, variant=9),
             lambda: binding.gcoo_from_csr(w.m, w.k, *dev, 0, known_nnz=True), lambda: binding.gcoo_from_csr(w.m, w.k, *dev, 257), lambda: binding.gcoo_from_csr(-1, w.k, *dev, 32),
             lambda: binding.gcoo_from_csr(w.m, w.k, dev[0].long(), *dev[1:], 32), lambda: binding.gcoo_from_csr(w.m, w.k, *[x.cpu() for x in dev], 32),
             lambda: binding.gcoo_from_csr(w.m, w.k, w.row_ptr, bad, w.vals, 32), lambda: binding.gcoo_from_csr(w.m, w.k, w.row_ptr[:-1], w.col_idx, w.vals, 0),
             lambda: binding.gcoo_from_dense(B.t(), 32), lambda: binding.gcoo_from_dense(B, 300), lambda: binding.gcoo_from_dense(B.half(), 32),
             lambda: binding.gcoo_from_csr_device_static(w.m, w.k, *dev, 32, out_buf=torch.empty(256, dtype=torch.uint8, device=DEV))]
    out = []
    for i, call in enumerate(calls):
        with pytest.raises((AssertionError, binding.GcooError, ValueError)) as e:
            call()
        out.append((i, e.type, str(e.value) if e.type is not AssertionError else ""))
    return out


def test_refuses_the_same_with_and_without_the_module(monkeypatch):
    w = workloads.uniform_random(120, 90, 40, 0.9, seed=4)
    dev = [torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)]
    by_module = _refused(w, dev)
    monkeypatch.setattr(binding, "_calls", _Nothing())
    assert by_module == _refused(w, dev)
