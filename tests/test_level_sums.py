"""Host check of the level launches' Z-type sums (no GPU needed): compiles
tests/level_sums_check.cpp, which runs the kernel's code with a host thread
per lane, and runs it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")


@pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm clang++ not installed")
def test_tiles_without_index_0_leave_zero_sums(tmp_path):
    exe = str(tmp_path / "level_sums_check")
    cmd = [CLANG, "-x", "c++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-w",
           "-I" + os.path.join(ROCM, "include"), "-I" + os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "level_sums_check.cpp"), "-o", exe, "-pthread"]
    b = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout[-4000:]
    assert "fails 0" in r.stdout
