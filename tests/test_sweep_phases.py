"""Host check of the phases of coupled blocks in sweeps (no GPU needed):
compiles tests/sweep_phases_check.hip, which includes the library's
sv_sweep.hip, and runs it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_phases_of_coupled_blocks(tmp_path):
    exe = str(tmp_path / "sweep_phases_check")
    cmd = [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I" + os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "sweep_phases_check.hip"), "-o", exe]
    b = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "fails 0" in r.stdout, r.stdout[-4000:]
