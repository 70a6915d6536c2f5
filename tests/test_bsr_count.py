"""The block-sparse symbolic count kernel with a scalar step beside it,
emulated on the CPU (bsr_count_check.cpp): uniform branches whatever the
waves read of a flag that is being set, and exact counts."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_waves_of_a_row_take_one_branch(tmp_path):
    src = open(os.path.join(ROOT, "paper_1507_02087_amd", "csrc", "bsr.hip")).read()
    start = src.index("constexpr int kCountThreads")
    end = src.index("\n}\n", src.index("void bsr_symbolic_count_kernel(", start)) + 3
    (tmp_path / "count_kernel.inc").write_text(src[start:end])
    exe = str(tmp_path / "bsr_count_check")
    b = subprocess.run(["g++", "-O1", "-std=c++20", "-pthread", "-I", str(tmp_path),
                        os.path.join(ROOT, "tests", "bsr_count_check.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    assert r.stdout.strip() == "ok"
