"""Which batches take the resident run (batch_rule_check.cpp, on the CPU), and
the teams of those that work through a list (run_list_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None,
                    reason="hipcc not available")
@pytest.mark.parametrize("check", ["batch_rule_check", "run_list_check"])
def test_host_check(tmp_path, check):
    exe = str(tmp_path / check)
    csrc = os.path.join(ROOT, "paper_1507_02087_amd", "csrc")
    b = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950",
                        "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(ROOT, "tests", check + ".cpp"),
                        "-x", "hip", os.path.join(csrc, "host_plan.hip"), "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert r.stdout.strip() == "ok"
