"""The transforms of a gate on twelve wavefronts (N = 1024), emulated on the host (CPU only): exchange slots, layouts
against the transform's definition, inverse round trip (tests/host_checks/quarter_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_quarter_transforms_on_the_host(tmp_path):
    from paper_1906_00148_amd import build as B
    exe = str(tmp_path / "quarter_check")
    subprocess.check_call([B.HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-ffp-contract=off",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", B.CSRC,
                           os.path.join(ROOT, "tests", "host_checks", "quarter_check.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout + r.stderr
