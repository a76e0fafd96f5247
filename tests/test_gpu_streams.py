"""Memory that the binding allocates and uses on a stream that the caller names: dropped while that stream is still at work, it is not given out again before
the stream has come to it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import gcoo_oracle as orc
from paper_2005_14469_amd import binding, workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_memory_used_on_another_stream_is_not_given_out_again():
    print("streams: memory dropped behind a busy stream", flush=True)
    w = workloads.uniform_random(900, 1100, 260, 0.95, seed=3)
    csr = [torch.from_numpy(x).to(DEV) for x in (w.row_ptr, w.col_idx, w.vals)]
    B = torch.from_numpy(w.B).to(DEV)
    kept = binding.gcoo_from_csr(w.m, w.k, *csr, 32, known_nnz=True)
    big, copy = torch.randn((4096, 4096), device=DEV), torch.empty((4096, 4096), device=DEV)
    want, C64, D64 = orc.gcoo_from_csr(w.m, w.k, w.row_ptr, w.col_idx, w.vals, 32), *orc.spdm_csr(w.k, w.N, w.row_ptr, w.col_idx, w.vals, w.B)
    st = torch.cuda.Stream(device=DEV)
    torch.cuda.synchronize()
    for call in ("csr", "static", "handle", "result"):
        with torch.cuda.stream(st):
            for _ in range(200):                               # some milliseconds, so that what follows on the stream is still to come when its memory is dropped
                copy.copy_(big)
        if call == "handle":
            C = torch.empty((w.m, w.N), device=DEV)
            binding.gcoo_spdm(kept, B, C, stream=st)
            size, at = kept.buf.numel(), kept.buf.data_ptr()
            kept.free()
        elif call == "result":
            C = binding.gcoo_spdm(A, B, stream=st)
            size, at = C.numel() * 4, C.data_ptr()
            del C
        else:
            make = (lambda **kw: binding.gcoo_from_csr(w.m, w.k, *csr, 32, known_nnz=True, **kw)) if call == "csr" else \
                   (lambda **kw: binding.gcoo_from_csr_device_static(w.m, w.k, *csr, 32, **kw))
            A = make(stream=st)
            size, at = A.buf.numel(), A.buf.data_ptr()
            A.free()
        busy = not st.query()
        again = torch.empty(size, dtype=torch.uint8, device=DEV)
        again.fill_(0x5a)                                      # on the current stream, at once
        assert busy and again.data_ptr() != at, call
        torch.cuda.synchronize()
        if call == "handle":
            err, bad = orc.max_scaled_error(C.cpu().numpy(), C64, D64)
            assert bad == 0 and err <= 1e-5
        A = binding.gcoo_from_csr(w.m, w.k, *csr, 32, known_nnz=True, stream=st)
        st.synchronize()
        e = A.export()
        assert np.array_equal(e["values"].view(np.uint32), want.values.view(np.uint32)) and np.array_equal(e["cols"], want.cols)
        del again
    with pytest.raises(ValueError, match="freed"):
        binding.gcoo_spdm(kept, B, stream=st)
