"""Host check of a sweep's descriptor loads (no GPU needed): compiles
tests/sweep_alignment_check.cpp, which runs the kernel's code with a host
thread per lane, with the alignment sanitizer, and runs it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CLANG = os.path.join(ROCM, "llvm", "bin", "clang++")


@pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm clang++ not installed")
def test_descriptors_are_read_at_their_alignment(tmp_path):
    exe = str(tmp_path / "sweep_alignment_check")
    cmd = [CLANG, "-x", "c++", "-std=c++17", "-O1", "-fsanitize=alignment", "-fno-sanitize-recover=alignment",
           "-D__HIP_PLATFORM_AMD__", "-w", "-I" + os.path.join(ROCM, "include"), "-I" + os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "sweep_alignment_check.cpp"), "-o", exe, "-pthread"]
    b = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "passed" in r.stdout, (r.returncode, r.stderr[-2000:])
