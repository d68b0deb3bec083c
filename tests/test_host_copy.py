"""The copies of device memory to the host (csrc/host_copy.hpp), driven on the CPU over a
stand-in for the runtime's entry points (host/copy_driver.cpp): many pieces and more of
them than one stage holds, pieces beside large ones, and pinned memory that is refused."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


@pytest.mark.skipif(not os.path.exists(os.path.join(HIP_INCLUDE, "hip", "hip_runtime_api.h")), reason="no HIP headers")
def test_pieces_arrive_whole(tmp_path):
    exe = tmp_path / "copy_driver"
    r = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-I", ROOT,
                        "-I", HIP_INCLUDE, os.path.join(ROOT, "tests", "host", "copy_driver.cpp"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "0 failures" in r.stdout, r.stdout[-3000:]
