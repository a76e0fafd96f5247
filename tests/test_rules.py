"""Rules of the library that are plain functions of sizes, compiled for the host."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rules") / "rules.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           os.path.join(ROOT, "tests", "host", "rules.cpp"), "-o", out])
    lib = C.CDLL(out)
    lib.band_tests.argtypes = [C.c_int32]
    lib.band_test_from.restype, lib.band_test_from.argtypes = C.c_int64, [C.c_int64, C.c_int32]
    lib.band_test_says.argtypes = [C.c_int64, C.c_int32]
    return lib


@pytest.mark.parametrize("lists", [1, 16, 255, 256, 257, 1023, 1024, 1025, 1280, 1281, 2672, 16672, 133360])
def test_lists_looked_at_grow_with_the_lists(rules, lists):
    """Every workgroup of a launch of that many (half as many where a workgroup has two lists) looks at 1024 at the most, and those that say what they find have looked at every list."""
    assert 1 <= rules.band_tests(lists) <= 1024
    for workgroups in (lists, (lists + 1) // 2):
        seen = np.zeros(lists + 1024, int)
        for w in range(workgroups):
            at = rules.band_test_from(w, lists)
            assert 0 <= at < lists
            if rules.band_test_says(w, lists):
                seen[at:at + rules.band_tests(lists)] += 1
        assert (seen[:lists] == 1).all()
