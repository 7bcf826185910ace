"""Host check of the multi-block sweeps' plan and index arithmetic (no GPU
needed): compiles tests/sweep_plan_check.hip, which includes the library's
sv_sweep.hip, and runs it over random programs on 1-36 qubits."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_sweep_plans_keep_order_and_cover_the_state(tmp_path):
    exe = str(tmp_path / "sweep_plan_check")
    csrc = os.path.join(ROOT, "paper_2308_01999_amd", "csrc")
    cmd = [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
           os.path.join(ROOT, "tests", "sweep_plan_check.hip"), "-o", exe]
    b = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(r.stdout)
    assert r.returncode == 0, r.stdout[-4000:]
    assert "fails 0" in r.stdout
