"""The LDS-resident levels' records on the host (CPU only): no cell without a thread, no
LDS image larger than a workgroup may use."""
import os
import shutil
import subprocess

import pytest


def test_every_cell_has_a_thread(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    lib = os.path.join(root, "paper_2106_03583_amd")
    exe = str(tmp_path / "coarse_host_driver")
    cmd = [hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(root, "include"), "-I", os.path.join(lib, "csrc"), "-x", "hip",
           os.path.join(root, "tests", "sanitize", "coarse_host_driver.cpp"), "-o", exe,
           "-L", lib, "-l:libmbp.so", f"-Wl,-rpath,{lib}"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "OK (0 failures" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
