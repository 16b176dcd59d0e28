"""How a launch is divided among the forms of the mixed blind rotation, on the host (CPU only): every gate exactly once
(tests/host_checks/mixed_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_gate_is_in_one_form(tmp_path):
    from paper_1906_00148_amd import build as B
    exe = str(tmp_path / "mixed_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(B.HIPCC))), "include"),
                           "-I", B.CSRC, os.path.join(ROOT, "tests", "host_checks", "mixed_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout + r.stderr
