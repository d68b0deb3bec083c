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


def test_checkpoint_leaves_the_callers_mapping_alone(rw, monkeypatch):
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
    # the Python call's own 7.7 MB may lie among other blocks: faulted in, not marked
    asked, real = [], rw._madvise
    monkeypatch.setattr(rw, "_madvise", lambda lo, size, advice: (asked.append((lo, size, advice)), real(lo, size, advice))[1])
    blob = rw.rewl_checkpoint(gpu.h)
    at = ctypes.cast(ctypes.c_char_p(blob), ctypes.c_void_p).value
    assert m[: n.value] == blob
    assert [a for _, _, a in asked] == [rw._POPULATE_WRITE]
    assert all(at <= lo and lo + size <= at + len(blob) and lo % 4096 == size % 4096 == 0 for lo, size, _ in asked)
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


def spans(kw, c):
    """Name and bytes of every piece of an instance's checkpoint, in their order."""
    W, WB = O.n_bins(c), int((O.layout(c)[1] - O.layout(c)[0]).max()) + 1
    L, h, m = kw["L"], kw["n_windows"], kw["m"]
    S, lattice = h * m, L * ((L + 63) // 64) * 8 if kw["model"] == "ising" else L * L
    return [("lattice", S * lattice), ("bins", S * 4), ("H", S * WB * 8), ("base", h * WB * 8), ("k", h * 4), ("done", h * 4), ("flat", S),
            ("swaps", S), ("ex_prop", h * 8), ("ex_acc", h * 8), ("merges", h * 4), ("rid", S * 4), ("rt_state", S), ("rt_count", S * 4),
            ("counters", 40)]


MIXED = ([dict(model="ising", L=8, n_windows=4, m=2)] * 20                       # pieces of a few bytes
         + [dict(model="ising", L=16, n_windows=8, m=8)] * 38                    # counts of 48 KB: 1.8 MB of small pieces
         + [dict(model="potts", q=10, L=16, n_windows=4, m=4)] * 5
         + [dict(model="potts", q=10, L=32, n_windows=8, m=256)]                 # counts of 12 MB, lattices of 2 MB
         + [dict(model="ising", L=66, n_windows=8, m=4), dict(model="ising", L=10, n_windows=3, m=1)])


def test_checkpoint_of_a_mixed_batch(rw):
    kws = [dict(kw, kfinal=8, X=60, seed=700 + i) for i, kw in enumerate(MIXED)]
    gpu = rw.Rewl([rw.make_config(**kw) for kw in kws])
    gpu.run(4)
    blob = rw.rewl_checkpoint(gpu.h)
    at, small = 16, 0
    assert np.frombuffer(blob[:16], np.uint64).tolist() == [0x4c57455232, len(kws)]
    for i, kw in enumerate(kws):
        st, ct, c = gpu.state(i), gpu.stats(i), O.make_config(**kw)
        p = {}
        for name, n in spans(kw, c):
            p[name] = np.frombuffer(blob[at: at + n], np.uint8)
            at += n
            small += n if n <= 65536 else 0
        S, N, L = kw["n_windows"] * kw["m"], kw["L"] ** 2, kw["L"]
        if kw["model"] == "potts":
            assert np.array_equal(p["lattice"].reshape(S, N), st["spins"])
        else:
            bits = np.unpackbits(p["lattice"].reshape(S, L, -1), axis=2, bitorder="little")[:, :, :L]
            assert np.array_equal(bits.reshape(S, N), st["spins"])
        for name, dtype, ref in (("bins", np.int32, st["bins"]), ("H", np.int64, st["H"].ravel()), ("k", np.int32, st["k"]),
                                 ("done", np.int32, st["done"]), ("flat", np.uint8, st["flat"]), ("swaps", np.int8, st["swaps"]),
                                 ("ex_prop", np.int64, ct["ex_prop"]), ("ex_acc", np.int64, ct["ex_acc"]),
                                 ("rt_count", np.int32, ct["round_trips"])):
            assert np.array_equal(p[name].view(dtype), ref), (i, name)
        base = np.repeat(p["base"].view(np.float64).reshape(kw["n_windows"], -1), kw["m"], axis=0)
        scale = np.repeat(2.0 ** -st["k"].astype(np.float64), kw["m"])[:, None]
        assert np.array_equal((st["H"] * scale + base).view(np.uint64), st["lng"].view(np.uint64))
        assert p["counters"].view(np.int64)[:2].tolist() == [4, ct["slow_decisions"]] and st["t"] == 4
        assert np.array_equal(np.sort(p["rid"].view(np.int32)), np.arange(S))
    assert at == len(blob) and small > 1 << 20
    # a fresh handle takes it up, and both go on alike, as the oracle does
    other = rw.Rewl([rw.make_config(**kw) for kw in kws])
    rw.rewl_restore(other.h, blob)
    assert rw.rewl_checkpoint(other.h) == blob
    gpu.run(5)
    other.run(5)
    assert rw.rewl_checkpoint(other.h) == rw.rewl_checkpoint(gpu.h) != blob
    for i in (0, 21, 57, 59, 64, 65):
        orc = O.Sim(O.make_config(**kws[i]))
        orc.run(9)
        assert_same(other.state(i), orc.state(), f"instance {i}")
    gpu.close()
    other.close()
