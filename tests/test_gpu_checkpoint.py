"""Checkpoints: memory that the caller owns stays as it is but for its bytes, and a batch
of many unequal instances is saved piece by piece, restored and continued bit for bit."""
import ctypes
import mmap

import numpy as np
import pytest

import oracle as O
from test_gpu_parity import assert_same, rw  # noqa: F401  (rw: fixture)

pytestmark = pytest.mark.gpu


def flags_at(address):
    """VmFlags of the mapping that holds the address, or None where nothing is mapped."""
    inside = False
    with open("/proc/self/smaps") as f:
        for line in f:
            head = line.split()[0]
            if "-" in head and not head.endswith(":"):
                lo, hi = (int(v, 16) for v in head.split("-"))
                inside = lo <= address < hi
            elif inside and head == "VmFlags:":
                return line.split()[1:]
    return None


def test_checkpoint_leaves_the_callers_mapping_alone(rw):
    gpu = rw.Rewl([rw.make_config(model="ising", L=64, n_windows=16, m=64, X=50, kfinal=12)])
    gpu.run(1)
    n = ctypes.c_size_t(0)
    assert rw._lib.rewl_checkpoint(gpu.h, None, ctypes.byref(n)) == rw.REWL_OK
    assert n.value > 6 << 20
    m = mmap.mmap(-1, n.value + (4 << 20))
    at = ctypes.addressof(ctypes.c_char.from_buffer(m))
    before = flags_at(at + (3 << 20))
    assert rw._lib.rewl_checkpoint(gpu.h, ctypes.c_void_p(at), ctypes.byref(n)) == rw.REWL_OK
    assert flags_at(at + (3 << 20)) == before and "hg" not in before
    blob = rw.rewl_checkpoint(gpu.h)
    assert m[: n.value] == blob
    where = ctypes.cast(ctypes.c_char_p(blob), ctypes.c_void_p).value + (3 << 20)
    assert "hg" not in flags_at(where)                       # nor does this one of 7.7 MB keep a mark
    gpu.close()


def test_large_checkpoint_takes_its_mapping_with_it(rw):
    gpu = rw.Rewl([rw.make_config(model="potts", q=10, L=64, n_windows=32, m=128, X=20, kfinal=12)])
    gpu.run(1)
    blob = rw.rewl_checkpoint(gpu.h)
    assert len(blob) > 40 << 20
    where = ctypes.cast(ctypes.c_char_p(blob), ctypes.c_void_p).value + (5 << 20)
    del blob
    assert "hg" not in (flags_at(where) or [])
    gpu.close()
