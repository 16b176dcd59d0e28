"""The half transforms (N = 1024, four points per lane) of the HIP library, emulated on the host (CPU only): exchange
slots, layout against the transform's definition, inverse round trip (tests/host_checks/half_check.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_half_transforms_on_the_host(tmp_path):
    from paper_1906_00148_amd import build as B
    exe = str(tmp_path / "half_check")
    subprocess.check_call([B.HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-ffp-contract=off",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", B.CSRC,
                           os.path.join(ROOT, "tests", "host_checks", "half_check.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "failures 0" in r.stdout, r.stdout + r.stderr
