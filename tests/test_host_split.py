"""The key switch's split of the coefficient range, on the host (CPU only): what the kernel takes, and close to the best of
the measured times at several key lengths (tests/host_checks/split_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_split_is_close_to_the_best_measured(tmp_path):
    from paper_1906_00148_amd import build as B
    exe = str(tmp_path / "split_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(B.HIPCC))), "include"),
                           "-I", B.CSRC, os.path.join(ROOT, "tests", "host_checks", "split_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout + r.stderr
