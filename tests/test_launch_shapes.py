"""Grids of every entry point over its documented range of sizes, recorded on the host (tests/host_sanitize/
launch_shapes.cpp): no dimension of a launch reaches 2^32 work-items, where a dispatch would run only a part of it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_launch_reaches_the_limit_of_a_dispatch(tmp_path):
    from paper_2411_08446_amd import build
    objs = [os.path.join(build.BUILD_DIR, os.path.splitext(s)[0] + ".o") for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        build.build(verbose=False)
    exe = str(tmp_path / "launch_shapes")
    obj = exe + ".o"
    src = os.path.join(ROOT, "tests", "host_sanitize", "launch_shapes.cpp")
    res = subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", "-c", src, "-o", obj], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([build.HIPCC, "--offload-arch=gfx950", obj, *objs, "-o", exe], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    assert " 0 failures" in res.stdout
