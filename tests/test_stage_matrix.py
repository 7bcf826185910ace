"""Host check of the matrix ring (no GPU needed): compiles
tests/stage_matrix_check.cpp, which includes the library's sv_api.cpp, and
runs it on buffers that end at an inaccessible page."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_staging_reads_no_byte_behind_the_buffer(tmp_path):
    obj, exe = str(tmp_path / "check.o"), str(tmp_path / "check")
    compile_cmd = [HIPCC, "-O1", "-std=c++17", "--offload-host-only", "-w", "-I" + os.path.join(ROOT, "include"), "-c",
                   "-x", "hip", os.path.join(ROOT, "tests", "stage_matrix_check.cpp"), "-o", obj]
    b = subprocess.run(compile_cmd, capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-4000:]
    # the file defines the HIP calls that staging makes; nothing else is reached
    link_cmd = ["g++", "-no-pie", obj, "-o", exe, "-Wl,--unresolved-symbols=ignore-all"]
    link = subprocess.run(link_cmd, capture_output=True, text=True, timeout=600)
    assert link.returncode == 0, link.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "passed" in r.stdout, (r.returncode, r.stdout)
