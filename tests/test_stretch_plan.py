"""The rules by which rows are dealt by columns (csrc/stretch.h), on the host (tests/host_sanitize/stretch_plan.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rules_of_rows_by_columns(tmp_path):
    from paper_2411_08446_amd import build
    exe = str(tmp_path / "stretch_plan")
    src = os.path.join(ROOT, "tests", "host_sanitize", "stretch_plan.cpp")
    res = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", src, "-o", exe], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    assert " 0 failures" in res.stdout
