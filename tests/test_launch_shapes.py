"""The launches of a time step, recorded instead of run (no GPU needed): the
library's launchers are called by tests/host/launch_shapes.cpp, which defines
hipLaunchKernel itself and checks the grids and workgroups handed to it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LIB_DIR = os.path.join(ROOT, "paper_2412_06546_amd")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_launch_shapes(tmp_path):
    lib = os.path.join(LIB_DIR, "libugks.so")
    if not os.path.exists(lib):
        from paper_2412_06546_amd import build
        build.build(force=False)
    exe = str(tmp_path / "launch_shapes")
    cmd = [HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", "-rdynamic",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(LIB_DIR, "csrc"), "-o", exe, "-x", "hip",
           os.path.join(ROOT, "tests", "host", "launch_shapes.cpp"), "-x", "none",
           "-L", LIB_DIR, "-l:libugks.so", "-Wl,-rpath," + LIB_DIR, "-ldl"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and " 0 failed" in r.stdout, (r.stdout + r.stderr)[-4000:]
    assert int(r.stdout.split()[0]) >= 200, r.stdout
