"""The ids that small CMux levels hand to the device in the kernel's arguments, on the host (CPU only): the lists, and nothing
of the host's memory beside them (tests/host_checks/cmux_ids_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_block_of_ids_holds_nothing_else(tmp_path):
    from paper_1906_00148_amd import build as B
    exe = str(tmp_path / "cmux_ids_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(B.HIPCC))), "include"),
                           "-I", B.CSRC, os.path.join(ROOT, "tests", "host_checks", "cmux_ids_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout[-500:] + r.stderr
