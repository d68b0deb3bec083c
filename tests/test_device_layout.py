"""Layouts that the kernels rely on, checked by the compiler (host pass only, no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

SOURCE = """
#include "paper_1407_5140_amd/csrc/rewl_device.hpp"
using rewl::InstCtr;
// k_collect reads its sources 16 bytes at a time, and instance i's counters are element i of an array
static_assert(alignof(InstCtr) % 16 == 0, "");
static_assert(sizeof(InstCtr) % 16 == 0, "");
// the bytes of a checkpoint: t and slow, then six words
static_assert(offsetof(InstCtr, t) == 0 && offsetof(InstCtr, slow) == 8 && offsetof(InstCtr, all_done) == 16, "");
static_assert(offsetof(InstCtr, stopped) == 20 && offsetof(InstCtr, n_done) == 24 && offsetof(InstCtr, err) == 28, "");
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_counters_of_every_instance_are_aligned(tmp_path):
    src = tmp_path / "layout.hip"
    src.write_text(SOURCE)
    r = subprocess.run([HIPCC, "--offload-host-only", "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "-I", ROOT, str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
