"""The C ABI on a fake device (CPU only; tests/host_checks/memory_check.cpp): calls short of memory, scratch that grows."""
from test_host_client import run_on_fake_device


def test_memory_on_the_fake_device(tmp_path):
    run_on_fake_device("memory_check.cpp", tmp_path)
