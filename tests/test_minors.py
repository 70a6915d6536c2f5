"""The eigenvalue count of the resident spectral norm on the CPU
(minors_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_count_at_and_beside_eigenvalues(tmp_path):
    src = open(os.path.join(ROOT, "paper_1507_02087_amd", "csrc", "spectral_run.hip")).read()
    start = src.index("constexpr double kPadLink")
    end = src.index("\n}\n", src.index("int minors_below(", start)) + 3
    (tmp_path / "minors.inc").write_text(src[start:end])
    exe = str(tmp_path / "minors_check")
    b = subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", str(tmp_path),
                        os.path.join(ROOT, "tests", "minors_check.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert r.stdout.strip() == "ok"
