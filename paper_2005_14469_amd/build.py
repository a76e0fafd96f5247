"""Compile the HIP library (csrc/*.hip -> libgcoo.so) for gfx950 with hipcc.  No GPU is needed.

Every .hip file is one translation unit; they are compiled in parallel and linked into one
shared library.  The binding's extension module is built beside it, with g++.
"""
from __future__ import annotations

import glob
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgcoo.so")
# the CSR row-split routine the benchmark compares against: a library of its own, not part of the GCOO path
BASELINE_SRC = os.path.join(HERE, "csrc_baseline", "csr_baseline.hip")
BASELINE_LIB = os.path.join(HERE, "libgcoo_baseline.so")
# the binding's calls as an extension module of the interpreter (host code only)
CALLS_SRC = os.path.join(HERE, "csrc_python", "calls.cpp")
CALLS_LIB = os.path.join(HERE, "_calls.so")

# Packed fp32 VALU instructions are switched off for every kernel of this library.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument",
         "-Wno-inline-asm"]      # the index-mode asm statements name M0 as clobbered, which clang remarks on


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _deps():
    return sources() + glob.glob(os.path.join(CSRC, "*.hpp")) + [os.path.join(ROOT, "include", "gcoo.h"), BASELINE_SRC, CALLS_SRC,
                                                                  os.path.join(ROOT, "include", "gcoo_baseline.h")]


def stale() -> bool:
    built = (LIB, BASELINE_LIB, CALLS_LIB)
    if not all(os.path.exists(x) for x in built):
        return True
    t = min(os.path.getmtime(x) for x in built)
    return any(os.path.getmtime(f) > t for f in _deps())


def _checked(src: str) -> bool:
    """Sources whose generated code is verified by isa_check (kernels that issue loads from asm, that load straight to LDS next
    to the index mode, or whose workgroups hand words to each other without release and acquire)."""
    name = os.path.basename(src)
    return name.startswith("spdm_sched_v") or name in ("spdm_share.hip", "spdm_band.hip", "gcoo_api.hip")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
    extra = ["-save-temps=obj"] if _checked(src) else []      # keeps the device assembly next to the object
    subprocess.check_call(["hipcc", *FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", obj])
    return obj


def sched_kernel_names(stem: str):
    """Mangled name prefixes of the kernels in spdm_sched_v<V>[t].hip (t = the tall accumulator layout)."""
    v = stem.rsplit("v", 1)[1]
    if v.endswith("t"):                  # that layout has no workgroup-shared kernel
        return (f"_ZN4gcoo8acc_tall10spdm_schedILi{v[:-1]}E",)
    return (f"_ZN4gcoo7acc_std10spdm_schedILi{v}E", f"_ZN4gcoo7acc_std15spdm_sched_coopILi{v}E")


def verify_generated_code() -> None:
    """Refuse to link a library whose asm-issued loads are not provably safe.

    The register SpDM kernel keeps loads in flight behind the compiler's back; isa_check proves
    on the assembly that no instruction touches a register before a wait has covered its load.
    A compiler change (or a careless edit) that breaks this would read stale registers or, worse,
    use them as addresses, so the check is part of the build, not only of the tests.
    """
    from . import isa_check
    for src in sources():
        if not _checked(src):
            continue
        stem = os.path.basename(src)[:-4]
        asm = os.path.join(OBJ, f"{stem}-hip-amdgcn-amd-amdhsa-gfx950.s")
        text = open(asm).read()
        if stem == "spdm_share":
            verify_share_code(stem, text)
            continue
        if stem == "spdm_band":
            verify_band_code(stem, text)
            continue
        if stem == "gcoo_api":
            verify_count_code(stem, text)
            continue
        for kernel in sched_kernel_names(stem):
            regs, bad = isa_check.check(text, kernel)
            if not regs:
                raise RuntimeError(f"{stem}: no asm-issued loads found in {kernel} (check is blind)")
            if bad:
                raise RuntimeError(f"{stem} {kernel}: {len(bad)} instructions touch registers with a load in flight, e.g. {bad[:3]}")


def verify_share_code(stem: str, text: str) -> None:
    """The workgroup-shared kernel: no register spills, all 256 VGPRs (two waves per SIMD), every load that
    writes LDS sets M0 itself, and in front of every barrier a wait that leaves at most the six row loads of
    the band after next in flight."""
    from . import isa_check
    kernel = "_ZN4gcoo10spdm_share"
    if not isa_check.kernel_body(text, kernel):
        raise RuntimeError(f"{stem}: kernel {kernel} not found")
    loads, problems = isa_check.check_lds_loads(text, kernel, in_flight=6)
    if not loads:
        raise RuntimeError(f"{stem} {kernel}: no loads to LDS found (check is blind)")
    if problems:
        raise RuntimeError(f"{stem} {kernel}: {problems[:3]}")
    spills = [int(x) for x in re.findall(r"\.vgpr_spill_count:\s+(\d+)", text)]
    if len(spills) != 1 or any(spills):
        raise RuntimeError(f"{stem}: register spills {spills}")


def verify_band_code(stem: str, text: str) -> None:
    """The sixteen-wave kernel, its instances (four and two columns per lane): no register spills, 128 VGPRs at most (four waves per SIMD), every load
    that writes LDS sets M0 itself, nothing is in flight at a barrier, and its asm text writes the scalar registers that its clobber list names."""
    from . import isa_check
    instances = [(4, 0, 0), (4, 0, 1), (4, 1, 0), (4, 1, 1), (2, 0, 0), (2, 0, 1), (2, 1, 0)]
    for v, spread, late in instances:
        kernel = f"_ZN4gcoo9spdm_bandILi{v}ELb{spread}ELb{late}E"
        loads, problems = isa_check.check_lds_loads(text, kernel, asm_only=True)
        if loads < 15 or problems or isa_check.check_lds_loads(text, kernel)[0] != loads:
            raise RuntimeError(f"{stem} {kernel}: {loads} loads to LDS, {problems[:3]}")
        written, read = isa_check.asm_scalar_writes(text, kernel)
        if written != set(range(12, 32)) | set(range(36, 100)) | ({100} if v == 2 else set()) or not read:
            raise RuntimeError(f"{stem} {kernel}: scalar registers written {sorted(written)}, read {sorted(read)}")
    meta = text[text.index("amdhsa.kernels"):]
    for key, most in (("vgpr_spill_count", 0), ("sgpr_spill_count", 0), ("private_segment_fixed_size", 0), ("vgpr_count", 128)):
        got = [int(x) for x in re.findall(rf"\.{key}:\s+(\d+)", meta)]
        if len(got) != len(instances) or max(got) > most:
            raise RuntimeError(f"{stem}: {key} {got}")


def verify_count_code(stem: str, text: str) -> None:
    """The dense counts: their workgroups hand what they counted to the last of them by agent scope and waits (Handed and arrive() in
    gcoo_build_kernels.hpp); the masks, in pieces of 8 and 16 bytes, are for later launches."""
    from . import isa_check
    masks = ("global_store_dwordx2", "global_store_dwordx4")
    for kernel, plain in [(f"_ZN4gcoo17count_dense_totalILi{v}E", ()) for v in (1, 4)] + \
                         [(f"_ZN4gcoo18count_dense_blocksILi{v}ELb{m}E", masks if m else ()) for v in (1, 4) for m in (0, 1)]:
        arrivals, problems = isa_check.check_arrivals(text, kernel, plain)
        if arrivals != 2 or problems:
            raise RuntimeError(f"{stem} {kernel}: {arrivals} arrivals, {problems[:3]}")


def _build_calls() -> None:
    import sysconfig
    import torch
    torch_dir = os.path.dirname(torch.__file__)
    inc, lib = os.path.join(torch_dir, "include"), os.path.join(torch_dir, "lib")
    tmp = CALLS_LIB + f".tmp{os.getpid()}"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                           "-I", os.path.join(ROOT, "include"), "-isystem", sysconfig.get_paths()["include"], "-isystem", inc,
                           "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), CALLS_SRC, "-o", tmp,
                           "-L", lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", f"-Wl,-rpath,{lib}"])
    os.replace(tmp, CALLS_LIB)


def build(force: bool = True, jobs: int = 8) -> str:
    if force or stale():
        os.makedirs(OBJ, exist_ok=True)
        with ThreadPoolExecutor(max_workers=jobs + 1) as ex:
            calls = ex.submit(_build_calls)
            objs = list(ex.map(_compile, sources()))
            calls.result()
        verify_generated_code()
        tmp = LIB + f".tmp{os.getpid()}"
        subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
        os.replace(tmp, LIB)
        tmp = BASELINE_LIB + f".tmp{os.getpid()}"
        subprocess.check_call(["hipcc", *FLAGS, "-shared", "-I", os.path.join(ROOT, "include"), BASELINE_SRC, "-o", tmp])
        os.replace(tmp, BASELINE_LIB)
    return LIB


def build_host_sanitized(jobs: int = 8) -> str:
    """A checking build: the same sources with the address and undefined-behaviour sanitizers on the HOST
    code only (the device code is compiled as usual), as _build/san/libgcoo.so.  For one pass of the tests that
    need no GPU; the command is printed by `python -m paper_2005_14469_amd.build --host-sanitize`."""
    out_dir = os.path.join(OBJ, "san")
    os.makedirs(out_dir, exist_ok=True)
    san = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-omit-frame-pointer"]
    flags = [*FLAGS, "-g", "-Xarch_host", "-O1"]          # (the device code as usual: the asm statements leave a lower level too few registers)

    def one(src):
        obj = os.path.join(out_dir, os.path.basename(src)[:-4] + ".o")
        subprocess.check_call(["hipcc", *flags, *san, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", obj])
        return obj
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(one, sources()))
    lib = os.path.join(out_dir, "libgcoo.so")
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *san[:4], "-shared-libsan", "-o", lib, *objs])
    return lib


if __name__ == "__main__":
    import sys
    if "--host-sanitize" in sys.argv[1:]:
        lib = build_host_sanitized()
        rt = glob.glob("/opt/rocm/lib/llvm/lib/clang/*/lib/linux/libclang_rt.asan-x86_64.so")
        print(lib)
        print(f"run: GCOO_LIBRARY={lib} LD_PRELOAD={rt[0] if rt else '<libclang_rt.asan-x86_64.so>'} ASAN_OPTIONS=detect_leaks=0 "
              "UBSAN_OPTIONS=halt_on_error=1 python -m pytest tests/test_abi_host.py tests/test_host_calls.py -q")
    else:
        print(build())
