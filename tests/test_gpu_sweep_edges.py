"""The sweeps at the sizes where their inner structure could go wrong, against the
CPU oracle, bit for bit (integer state and ln g): intervals around the draw
chunks (4, 8 and 64 attempts), proposed states above 127 (byte comparisons), odd
and two-word rows, lattices smaller than a chunk (nearly every attempt is evaluated
again), and tables so steep that a walker leaves the range of the FP32 differences
at every other move, with every decision near its threshold taken exactly."""
import numpy as np
import pytest

import oracle as O
from test_gpu_parity import _tune, assert_same, rw  # noqa: F401  (rw: fixture)

pytestmark = pytest.mark.gpu

KINDS = ["lane", "lane-persist", "wave", "wave-device", "wave-map64"]


def lockstep(rw, kw, tune, calls, table=None):
    gpu, orc = rw.Rewl([rw.make_config(**kw)], tune=tune), O.Sim(O.make_config(**kw), init_lng=table)
    try:
        if table is not None:
            gpu.set_initial_lng(table)
        for n in calls:
            gpu.run(n)
            orc.run(n)
            assert_same(gpu.state(), orc.state(), f"{kw} after {orc.t} intervals")
        return gpu.stats()
    finally:
        gpu.close()


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("X", [1, 3, 4, 5, 7, 8, 9, 63, 64, 65, 130])
def test_intervals_around_the_chunks(rw, kind, X):
    for kw in (dict(model="ising", L=6, n_windows=2, m=2), dict(model="potts", q=5, L=7, n_windows=2, m=4)):
        lockstep(rw, dict(kw, kfinal=12, X=X, seed=300 + X), _tune(rw, kind), (1, 2, 20))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("kw", [dict(model="potts", q=200, L=9, n_windows=3, m=2), dict(model="potts", q=129, L=4, n_windows=1, m=2),
                                dict(model="ising", L=126, n_windows=8, m=1), dict(model="ising", L=66, n_windows=4, m=2),
                                dict(model="potts", q=3, L=65, n_windows=8, m=1), dict(model="ising", L=4, n_windows=1, m=64)],
                         ids=lambda kw: f"{kw['model']}{kw.get('q', 2)}-L{kw['L']}")
def test_shapes(rw, kind, kw):
    lockstep(rw, dict(kw, kfinal=12, X=1500, seed=411), _tune(rw, kind), (1, 3))


@pytest.mark.parametrize("kind", ["lane", "wave", "wave-device"])
@pytest.mark.parametrize("slope", [0.0, 7.0, 300.0])
@pytest.mark.parametrize("band", [0, -2])
def test_steep_tables_and_wide_band(rw, kind, slope, band):
    """ln g rising and falling by `slope` per bin (zigzag), at ln f = 1 and 2^-12."""
    t = _tune(rw, kind)
    t.guard_band_log2 = band
    for kw in (dict(model="ising", L=12, n_windows=2, m=2), dict(model="potts", q=10, L=10, n_windows=2, m=2)):
        N = kw["L"] ** 2
        W = N + 1 if kw["model"] == "ising" else 2 * N + 1
        table = slope * np.abs((np.arange(W) % 40) - 20.0)
        for k0 in (0, 12):
            st = lockstep(rw, dict(kw, k0=k0, kfinal=30, X=2000, seed=511), t, (1, 4), table)
            if band and slope == 0.0:
                assert st["slow_decisions"] > 0


@pytest.mark.parametrize("small,lanes", [(31, False), (32, True)])
def test_auto_splits_a_batch(rw, small, lanes):
    """15 872 and 16 384 walkers of small tables beside a larger lattice: the variant per
    instance, and the same states as with either variant for all."""
    kws = [dict(model="ising", L=6, n_windows=2, m=256, kfinal=12, X=70, seed=s) for s in range(small)]
    kws.insert(3, dict(model="potts", q=10, L=32, n_windows=3, m=2, kfinal=12, X=70, seed=99))
    states = []
    for kind in ("auto", "lane", "wave"):
        gpu = rw.Rewl([rw.make_config(**kw) for kw in kws], tune=rw.make_tune(kind))
        if kind == "auto":
            assert [gpu.info(i)["sweep_kind"] for i in (0, 3, small)] == (["lane", "wave", "lane"] if lanes else ["wave"] * 3)
        gpu.run(5)
        states.append([gpu.state(i) for i in (0, 3, small)])
        gpu.close()
    for other in states[1:]:
        for a, b in zip(states[0], other):
            assert_same(a, b, f"{small} small instances")


@pytest.mark.parametrize("use_graph", [0, 1])
def test_blocks_in_order_of_work(rw, use_graph):
    """More blocks than the GPU has CUs, of windows with unequal work: reordered on the device
    between the intervals, every walker swept once in each of them."""
    kw = dict(model="potts", q=10, L=8, n_windows=3, m=512, kfinal=12, X=130, seed=77)
    gpu = rw.Rewl([rw.make_config(**kw)], tune=rw.make_tune("wave", walkers_per_block=2, use_graph=use_graph))
    orc = O.Sim(O.make_config(**kw))
    assert gpu.info()["walkers_per_block"] == 2                          # 768 blocks
    for n in (1, 1, 8, 9):
        gpu.run(n)
        orc.run(n)
        assert_same(gpu.state(), orc.state(), f"after {orc.t} intervals")
    gpu.close()


@pytest.mark.parametrize("kind", ["lane", "lane-persist"])
@pytest.mark.parametrize("short", [0, 16, 64, 128, 160])
@pytest.mark.parametrize("kw", [dict(model="ising", L=128), dict(model="potts", q=10, L=100)],
                         ids=lambda kw: f"{kw['model']}-L{kw['L']}")
def test_lane_tables_that_fill_the_lds(rw, kind, short, kw):
    """One walker's table, counts and lattice take the 160 KiB of a block up to `short` bytes
    (and up to the queue's 16 bytes): its draws, 128 bytes, find room there or elsewhere."""
    L, N = kw["L"], kw["L"] ** 2
    W = N + 1 if kw["model"] == "ising" else 2 * N + 1
    lattice = L * ((L + 63) // 64) * 8 if kw["model"] == "ising" else N
    WB = min(W - 40, (163840 - 16 - short - lattice) // 12 - 8)
    kw = dict(kw, n_windows=2, m=2, kfinal=12, X=300, seed=611, windows=([0, WB - 30], [WB - 1, W - 1]))
    t = _tune(rw, kind)
    t.walkers_per_block = 1
    gpu = rw.Rewl([rw.make_config(**kw)], tune=t)
    info = gpu.info()
    gpu.close()
    assert info["sweep_kind"] == "lane" and info["walkers_per_block"] == 1 and info["lds_bytes"] <= 163840
    lockstep(rw, kw, t, (1, 2))


@pytest.mark.parametrize("instances,lds_kb,effect", [(2, 0, (0, 0)), (2, 53, (0, 53)), (64, 0, (1, 40)), (64, 53, (1, 53))])
def test_tune_reports_what_auto_uses(rw, instances, lds_kb, effect):
    import bench
    cfgs = [rw.make_config(model="ising", L=6, n_windows=2, m=256, kfinal=12, X=50, seed=s) for s in range(instances)]
    gpu = rw.Rewl(cfgs, tune=rw.make_tune("auto", lds_target_kb=lds_kb))
    tune, info = gpu.tune(), gpu.info()
    assert (tune["persistent"], tune["lds_target_kb"]) == effect and tune["sweep_kind"] == 0
    assert bench.sweep_kernel(info, tune) == ("k_sweep_persist" if instances == 64 else "k_sweep_wave")
    gpu.run(2)
    again = rw.Rewl(cfgs, tune=rw.rewl_tune(**tune))
    again.run(2)
    assert again.tune() == tune and again.info() == info
    assert_same(gpu.state(5 % instances), again.state(5 % instances), "created with the tuning in effect")
    gpu.close()
    again.close()


def test_lane_tiles_of_both_kinds_in_a_batch(rw):
    """Tiles with their draws in device memory beside ones with them in the LDS."""
    big = dict(model="potts", q=10, L=100, n_windows=2, m=2, windows=([0, 12781], [12810, 20000]))
    kws = [dict(kw, kfinal=12, X=300, seed=s) for s, kw in enumerate([dict(model="ising", L=8, n_windows=4, m=4), big, dict(model="potts", q=4, L=9, n_windows=2, m=8), big])]
    for persistent in (0, 1):
        gpu = rw.Rewl([rw.make_config(**kw) for kw in kws], tune=rw.make_tune("lane", walkers_per_block=4, persistent=persistent))
        assert gpu.info(1)["lds_bytes"] > 163840 - 128
        gpu.run(3)
        for i, kw in enumerate(kws):
            orc = O.Sim(O.make_config(**kw))
            orc.run(3)
            assert_same(gpu.state(i), orc.state(), f"instance {i}")
        gpu.close()


@pytest.mark.parametrize("kw,n,lane", [
    (dict(model="ising", L=8, n_windows=8, m=64), 32, True),                      # 16 384 walkers in tiles of 64
    (dict(model="ising", L=8, n_windows=8, m=64), 31, False),
    (dict(model="ising", L=8, n_windows=8, m=8), 256, True),                      # tiles of 8, few sites
    (dict(model="ising", L=8, n_windows=8, m=4), 512, False),                     # tiles of 4
    (dict(model="ising", L=16, n_windows=8, m=8), 300, False),                    # tiles of 8, more sites
    (dict(model="ising", L=16, n_windows=8, m=16), 140, True),                    # tiles of 16, 17 476 walkers needed
    (dict(model="ising", L=16, n_windows=8, m=16), 136, False),
    (dict(model="potts", q=10, L=16, n_windows=8, m=64), 54, False),              # 27 904 needed
    (dict(model="potts", q=10, L=16, n_windows=8, m=64), 55, True),
    (dict(model="potts", q=10, L=16, n_windows=8, m=1), 4096, False)],            # one walker to a tile
    ids=lambda v: f"{v['model']}-L{v['L']}-m{v['m']}" if isinstance(v, dict) else str(v))
def test_autos_choice(rw, kw, n, lane):
    """The variant that AUTO takes, and the states of the first and last instance."""
    kws = [dict(kw, kfinal=12, X=70, seed=s) for s in range(n)]
    gpu = rw.Rewl([rw.make_config(**kw) for kw in kws], tune=rw.make_tune("auto"))
    assert {gpu.info(i)["sweep_kind"] for i in range(n)} == {"lane" if lane else "wave"}
    gpu.run(3)
    for i in (0, n - 1):
        orc = O.Sim(O.make_config(**kws[i]))
        orc.run(3)
        assert_same(gpu.state(i), orc.state(), f"instance {i}")
    gpu.close()
