"""The C ABI on a fake device that runs out of memory (CPU only; tests/host_checks/memory_check.cpp)."""
from test_host_client import run_on_fake_device


def test_a_call_short_of_memory_leaves_no_error_behind(tmp_path):
    run_on_fake_device("memory_check.cpp", tmp_path)
