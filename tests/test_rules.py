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
    lib.rows_turn.argtypes = [C.c_int32, C.c_int64, C.c_int64]
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


@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 7, 9, 12])
@pytest.mark.parametrize("row_wgs", [1, 2, 3, 7, 8, 9, 40, 63, 64, 65, 1000, 1249, 65521, 65535])
def test_long_rows_are_dealt_to_the_xcds(rules, row_wgs, tiles):
    """Every place has one workgroup of a tile that begins with it, and where two or more XCDs come to a tile one of them begins with no more than three quarters of the first sixteen."""
    rest = tiles % 8
    turn = np.array([rules.rows_turn(wg, row_wgs, tiles) for wg in range(row_wgs)])
    assert sorted(turn) == list(range(row_wgs))
    per_xcd = -(-rest * row_wgs // 8)
    for tile in range(rest):
        xcd = (tile * row_wgs + np.arange(row_wgs)) // per_xcd
        first = np.bincount(xcd[turn < 16], minlength=8)
        if row_wgs >= 40 and rest <= 4:
            assert first.max() <= 12, (tile, first)
