"""The client's calls of the C ABI on a fake device (CPU only): what they leave behind (tests/host_checks/client_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHECKS = os.path.join(ROOT, "tests", "host_checks")
HOST_SOURCES = ["she_api.cpp", "she_host.cpp", "she_circuits.cpp", "she_leveled.cpp"]


def run_on_fake_device(check, tmp_path):
    """Builds `check` with the library's host files and without the HIP runtime, and runs it."""
    from paper_1906_00148_amd import build as B
    exe = str(tmp_path / "check")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-pthread", "-ffp-contract=off", "-w", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(B.HIPCC))), "include"),
                           "-I", B.CSRC] + [os.path.join(B.CSRC, s) for s in HOST_SOURCES] +
                          [os.path.join(CHECKS, check), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout + r.stderr


def test_client_calls_leave_no_secret_behind(tmp_path):
    run_on_fake_device("client_check.cpp", tmp_path)


def test_samples_are_read_without_device_memory_to_spare(tmp_path):
    run_on_fake_device("read_check.cpp", tmp_path)
