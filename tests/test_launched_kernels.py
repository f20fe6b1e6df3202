"""Kernels that the entry points launch, looked at on the host (tests/host_sanitize/launched_kernels.cpp):
no read of a caller's array beyond the entries that the header gives it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kernels_of_the_entry_points(tmp_path):
    from paper_2411_08446_amd import build
    objs = [os.path.join(build.BUILD_DIR, os.path.splitext(s)[0] + ".o") for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        build.build(verbose=False)
    exe = str(tmp_path / "launched_kernels")
    obj = exe + ".o"
    src = os.path.join(ROOT, "tests", "host_sanitize", "launched_kernels.cpp")
    res = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", "-c", src, "-o", obj], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([build.HIPCC, "--offload-arch=gfx950", obj, *objs, "-o", exe], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    assert " 0 failures" in res.stdout
