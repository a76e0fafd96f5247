"""The host code of the library without a GPU (see host_calls.py): one process per case."""
import subprocess
import sys

import pytest

from tests import host_calls


@pytest.fixture(scope="module", autouse=True)
def stub():
    host_calls.build()


@pytest.mark.parametrize("case", ["wide_pitch", "few_columns", "host_csr_under_capture", "counts_under_capture", "stage_release_fails", "starts_of_a_changing_input", "pinned_memory_is_coherent", "slot_wait_fails", "slot_launch_fails", "looks_before_waiting", "dense_waits", "dense_launches", "order_lds", "places_in_turns", "no_columns", "kernel_of_product", "tiles", "sums", "widths", "cuts", "requests", "tall_rounds", "parts_of_power_law_rows", "one_handle_many_threads"])
def test_host_code(case):
    r = subprocess.run([sys.executable, "-m", "tests.host_calls", case], cwd=host_calls.ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr
