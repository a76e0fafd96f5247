"""The work that a user of this framework has it do, as cases that can be timed.

C = A x B in fp32, A sparse.  A case names the matrix (m x k, its density or its row lengths), the width N of B and
the route, that is, what the program holds and calls:

  known   A is a CSR matrix on the device and the program knows its entry count: conversion to GCOO and one product
          (the step that bench.py times; a matrix that is multiplied once, or whose values change from step to step)
  read    the same without the count: the conversion reads it back
  static  the same through the conversion that allocates nothing, into a buffer that the program keeps
  dense   A is a dense matrix on the device: count, conversion (Algorithm 1) and one product
  host    A is a CSR matrix in host memory (scipy's arrays): copy, conversion and one product
  kept    A was converted before: one product (an iterative solver, a layer with fixed weights)

The matrices are the ones of the paper's evaluation as far as they can be drawn: cells placed uniformly at random,
n between 400 and 14000, sparsity between 0.8 and 0.9995 (Section 4.2), power-law row lengths for the skewed ones
(the fifth configuration in workloads.py), N(0,1) values.  Group heights are the library's default for the shape.
"""
import math

import numpy as np
import torch

from paper_2005_14469_amd import binding

DEV = "cuda:0"
ZIPF_EXPONENT, ZIPF_ROW_MAX = 1.5, 4096      # row lengths of the skewed matrices, as in workloads.zipf_rows
MOST_PRODUCTS = 5.5e10                       # stored entries x N of the largest case


def listed():
    return [
        # the smallest step: the first configuration of workloads.py, where launches and the host path are all there is
        dict(name="step_256", route="known", rows="uniform", m=256, k=256, N=256, density=0.1),
        # the smallest matrix of the paper's random set, multiplied again and again
        dict(name="kept_400", route="kept", rows="uniform", m=400, k=400, N=400, density=0.02),
        # nothing square, nothing a multiple of anything, entry count unknown to the caller
        dict(name="ragged_1777", route="read", rows="uniform", m=1777, k=2301, N=1117, density=0.03),
        # an ordinary matrix that arrives from host memory
        dict(name="host_2500", route="host", rows="uniform", m=2500, k=2500, N=1024, density=0.01),
        # Algorithm 1 from a dense matrix, n = 4000 as in Section 4.3
        dict(name="dense_4000", route="dense", rows="uniform", m=4000, k=4000, N=4000, density=0.02),
        # the second configuration of workloads.py
        dict(name="step_4000", route="known", rows="uniform", m=4000, k=4000, N=4000, density=0.05),
        # the fourth one: the headline workload of bench.py
        dict(name="step_8000_sparse", route="known", rows="uniform", m=8000, k=8000, N=8000, density=0.005),
        # the third one: the case of the paper's introduction, the densest of the large ones
        dict(name="step_8000", route="known", rows="uniform", m=8000, k=8000, N=8000, density=0.1),
        # the sparse end of the paper's range, with an odd size
        dict(name="step_12001_sparsest", route="known", rows="uniform", m=12001, k=12001, N=12001, density=0.0005),
        # the fifth configuration: power-law row lengths, through the conversion that allocates nothing
        dict(name="skewed_16384", route="static", rows="zipf", m=16384, k=16384, N=512),
        # a narrow B: a block of vectors of an iterative method, features of a graph's nodes
        dict(name="narrow_12000", route="kept", rows="uniform", m=12000, k=12000, N=64, density=0.005),
        # the largest size of the paper's sweeps
        dict(name="kept_14000", route="kept", rows="uniform", m=14000, k=14000, N=14000, density=0.02),
    ]


def _spread(rng, lo, hi):
    """A number between lo and hi, spread over its logarithm."""
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _around(rng, n, most):
    """A size near n: n itself half the time, else anything from 0.6 n to 1.6 n."""
    return n if rng.random() < 0.5 else max(1, min(most, int(n * rng.uniform(0.6, 1.6))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "kept", "kept", "narrow", "skewed", "dense", "host"])
    if kind == "skewed":
        m = int(_spread(rng, 2000, 20000))
        return dict(route=rng.choice(["known", "read", "static", "kept"]), rows="zipf", m=m, k=_around(rng, m, 20000),
                    N=int(_spread(rng, 64, 1024)))
    if kind == "narrow":
        m = int(_spread(rng, 1000, 20000))
        return dict(route=rng.choice(["kept", "known"]), rows="uniform", m=m, k=_around(rng, m, 20000), N=int(_spread(rng, 16, 256)),
                    density=round(_spread(rng, 0.0005, 0.02), 6))
    if kind == "host":
        m = int(_spread(rng, 256, 4000))
        k = _around(rng, m, 4000)
        return dict(route="host", rows="uniform", m=m, k=k, N=int(_spread(rng, 256, 4000)),
                    density=round(min(_spread(rng, 0.0005, 0.2), 3e5 / (m * k)), 6))
    n = int(_spread(rng, 256, 14000))
    if kind == "dense":
        n = min(n, 8000)
    m, k, N = (_around(rng, n, 14500) for _ in range(3))
    density = min(_spread(rng, 0.0005, 0.2), MOST_PRODUCTS / (m * k * N))
    route = {"step": rng.choice(["known", "known", "read", "static"]), "kept": "kept", "dense": "dense"}[kind]
    if route == "static" and density * m * k > binding.GCOO_STATIC_MAX_NNZ:
        route = "known"
    return dict(route=route, rows="uniform", m=m, k=k, N=N, density=round(max(density, 1e-6), 6))


def _csr_from_cells(cells, m, k, g):
    """CSR arrays on the device from ascending cell numbers (row * k + column), with N(0,1) values."""
    rows = torch.div(cells, k, rounding_mode="floor")
    row_ptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=m), 0)
    vals = torch.randn(cells.numel(), generator=g, device=DEV, dtype=torch.float32)
    return row_ptr.to(torch.int32), (cells - rows * k).to(torch.int32), vals


def _uniform_csr(case, g):
    """Exactly round(density * m * k) cells, drawn without replacement."""
    m, k = case["m"], case["k"]
    want = _entries(case)
    cells = torch.empty(0, dtype=torch.int64, device=DEV)
    while cells.numel() < want:
        more = torch.randint(m * k, (int(1.2 * (want - cells.numel())) + 64,), generator=g, device=DEV)
        cells = torch.unique(torch.cat([cells, more]))
    keep = torch.randperm(cells.numel(), generator=g, device=DEV)[:want]
    return _csr_from_cells(torch.sort(cells[keep]).values, m, k, g)


def _zipf_csr(case, seed, g):
    """Power-law row lengths; the cells of a row are uniform over its columns."""
    m, k = case["m"], case["k"]
    rng = np.random.default_rng(seed)
    lens = rng.zipf(ZIPF_EXPONENT, size=m)
    while (lens > ZIPF_ROW_MAX).any():
        bad = lens > ZIPF_ROW_MAX
        lens[bad] = rng.zipf(ZIPF_EXPONENT, size=int(bad.sum()))
    share = torch.from_numpy(np.minimum(lens, k) / k).to(DEV, torch.float32)
    hit = torch.rand((m, k), generator=g, device=DEV) < share[:, None]
    return _csr_from_cells(hit.reshape(-1).nonzero().reshape(-1), m, k, g)


def _entries(case):
    """Stored entries of A: the count itself for uniform cells, its expectation for power-law rows."""
    if case["rows"] == "uniform":
        return max(1, int(round(case["density"] * case["m"] * case["k"])))
    x = np.arange(1, ZIPF_ROW_MAX + 1, dtype=np.float64)
    w = x ** -ZIPF_EXPONENT
    return int(case["m"] * (w * np.minimum(x, case["k"])).sum() / w.sum())


def prepare(case, seed):
    m, k, N, route = case["m"], case["k"], case["N"], case["route"]
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    state = dict(route=route, m=m, k=k)
    if route == "dense":
        keep = torch.rand((m, k), generator=g, device=DEV) < case["density"]
        state["A"] = torch.randn((m, k), generator=g, device=DEV) * keep
        state["p"] = binding.gcoo_default_p(m, k, _entries(case), N)
    else:
        csr = _uniform_csr(case, g) if case["rows"] == "uniform" else _zipf_csr(case, seed, g)
        nnz = int(csr[1].numel())
        p = state["p"] = binding.gcoo_default_p(m, k, nnz, N)
        if route == "kept":
            state["handle"] = binding.gcoo_from_csr(m, k, *csr, p, known_nnz=True)
            state["C"] = torch.empty((m, N), dtype=torch.float32, device=DEV)
        elif route == "host":
            state["csr"] = tuple(x.cpu().numpy() for x in csr)
        else:
            state["csr"] = csr
        if route == "static":
            state["buf"] = torch.empty(binding.lib().gcoo_static_handle_bytes(m, k, nnz, p), dtype=torch.uint8, device=DEV)
            state["C"] = torch.empty((m, N), dtype=torch.float32, device=DEV)
    state["B"] = torch.randn((k, N), generator=g, device=DEV, dtype=torch.float32)
    return state


def run(state):
    route, m, k, p, B = state["route"], state["m"], state["k"], state["p"], state["B"]
    if route == "kept":
        return binding.gcoo_spdm(state["handle"], B, state["C"])
    if route == "dense":
        A = binding.gcoo_from_dense(state["A"], p)
    elif route == "static":
        A = binding.gcoo_from_csr_device_static(m, k, *state["csr"], p, out_buf=state["buf"])
    else:
        A = binding.gcoo_from_csr(m, k, *state["csr"], p, device=DEV, known_nnz=route == "known")
    C = binding.gcoo_spdm(A, B, state.get("C"))
    A.free()
    return C


def work(case):
    m, k, N, nnz = case["m"], case["k"], case["N"], _entries(case)
    if case["route"] == "dense":
        a = 4.0 * m * k
    elif case["route"] == "kept":
        a = 12.0 * nnz                                  # values, rows, cols of the format
    else:
        a = 8.0 * nnz + 4.0 * (m + 1)                   # the CSR arrays
    # rows of B that a stored entry touches (all of them but for the sparsest matrices)
    touched = k * -math.expm1(-nnz / k) if case["rows"] == "uniform" else k
    return dict(bytes=a + 4.0 * touched * N + 4.0 * m * N, flops=2.0 * nnz * N)


def tolerance(case):
    return dict(rel=1e-5)                               # sums of 32-bit products in another order
