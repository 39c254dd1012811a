"""The attention kernels' tile order, on the CPU: heads go to one XCD each only
where the eight heads that run side by side have equal work, and every tile is
taken once."""
import os
import subprocess

from paper_2609_23169_amd import _build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_tile_order(tmp_path):
    exe = str(tmp_path / "check_tile_order")
    cmd = [_build.GXX, "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I", os.path.join(os.path.dirname(HERE), "include"), "-I", _build.CSRC,
           os.path.join(HERE, "host", "check_tile_order.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failure(s)" in r.stdout, r.stdout
