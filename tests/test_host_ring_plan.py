"""Host-side ring planning under AddressSanitizer and UndefinedBehaviorSanitizer
(CPU only): the complex128 Bluestein classes and their LDS, the layouts of
Delta, and how rings are dealt to the XCDs (tests/sanitize/ring_plan_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_ring_plan_under_sanitizers(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc missing")
    exe = str(tmp_path / "ring_plan_driver")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17",
                           "-Xarch_host", "-fsanitize=address,undefined",
                           "-Xarch_host", "-fno-sanitize-recover=all", "-g",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1010_1260_amd", "csrc"),
                           os.path.join(HERE, "sanitize", "ring_plan_driver.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "ring plan driver ok" in r.stdout
