"""The level scheduler on the host (CPU only): evened levels are right and no slower by the estimate
(tests/host_checks/levels_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_evened_levels(tmp_path):
    from paper_1906_00148_amd import build as B
    exe = str(tmp_path / "levels_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(B.HIPCC))), "include"),
                           "-I", B.CSRC, os.path.join(ROOT, "tests", "host_checks", "levels_check.cpp"),
                           os.path.join(B.CSRC, "she_circuits.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout + r.stderr
