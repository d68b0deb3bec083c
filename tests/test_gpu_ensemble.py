"""GPU parity of the n-run error analysis (rewl_ensemble) and of the canonical
averages (rewl_thermo) against the oracle.

Join points are integer decisions taken on bit-identical mean pieces (the sum
in run order and the division by n are single IEEE operations on both sides),
so they must match exactly; the joined ln g differs only in the normalisation's
exp/log (bound 1e-9, as for rewl_concat).  The canonical sums run in another
order and with another exp: relative differences stay near 1e-13, tested at
1e-10 (u, f) and 1e-9 (c, plus 1e-12 of the row's largest c for values that
vanish at low temperature).
"""
import numpy as np
import pytest

import oracle as O
from oracle import ensemble as EN

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rw():
    import paper_1407_5140_amd as rw
    return rw


def _assert_thermo(g, o):
    gu, gc, gf = g
    ou, oc, of = o
    assert np.all(np.abs(gu - ou) <= 1e-10 * np.maximum(1.0, np.abs(ou)))
    assert np.all(np.abs(gf - of) <= 1e-10 * np.maximum(1.0, np.abs(of)))
    cmax = np.max(oc, axis=1, keepdims=True)
    assert np.all(np.abs(gc - oc) <= 1e-9 * np.abs(oc) + 1e-12 * cmax)


def _oracle_thermo(model, L, rows, T):
    out = [EN.canonical(model, L, r, T) for r in rows]
    return tuple(np.array([o[k] for o in out]) for k in range(3))


T_GRID = np.concatenate([np.geomspace(0.05, 1e4, 45), np.linspace(2.1, 2.5, 16)])   # 61: ragged tile


@pytest.mark.parametrize("name,L", [("ising_L16_lng.txt", 16), ("ising_L64_lng.txt", 64)])
def test_thermo_parity_ising_exact_and_noisy(rw, golden, name, L):
    lg = golden.lng(name)
    rng = np.random.default_rng(L)
    rows = [lg, np.where(np.isfinite(lg), lg + rng.normal(0, 0.05, lg.size), -np.inf), lg + 1e3]
    g = rw.rewl_thermo("ising", L, np.array(rows), T_GRID)
    _assert_thermo(g, _oracle_thermo("ising", L, rows, T_GRID))


def test_thermo_parity_potts_exact(rw, golden):
    from oracle import exact_dos as X
    lg = X.ln_g(golden.counts("potts_q3_L5_counts.txt"))
    T = np.geomspace(0.05, 100.0, 9)                               # one full tile and one of 1
    g = rw.rewl_thermo("potts", 5, lg[None, :], T)
    _assert_thermo(g, _oracle_thermo("potts", 5, [lg], T))


def test_thermo_rejects_bad_input(rw):
    lg = np.zeros(17)
    with pytest.raises(rw.RewlError):
        rw.rewl_thermo("ising", 4, lg, [0.0])
    with pytest.raises(rw.RewlError):
        rw.rewl_thermo("ising", 4, np.full(17, -np.inf), [1.0])
    bad = lg.copy()
    bad[3] = np.nan
    with pytest.raises(rw.RewlError):
        rw.rewl_thermo("ising", 4, bad, [1.0])
    with pytest.raises(rw.RewlError):
        rw.rewl_thermo(2, 4, lg, [1.0])                     # no such model
    with pytest.raises(ValueError):
        rw.rewl_thermo("ising", 4, np.zeros(16), [1.0])     # rows must span the model's W bins


def _small_kws():
    return [dict(model="ising", L=8, n_windows=4, m=2, kfinal=12, X=1000, seed=s) for s in (1, 2, 3)]


def test_ensemble_of_converged_runs(rw):
    """Three independent runs to convergence (the oracle's own runs supply its
    pieces; lockstep parity makes the GPU's identical), mean + 24 resamples."""
    kws = _small_kws()
    gpu = rw.Rewl([rw.make_config(**kw) for kw in kws])
    for _ in range(400):
        if gpu.run(200):
            break
    runs = []
    for kw in kws:
        sim = O.Sim(O.make_config(**kw))
        assert sim.run(100000)
        runs.append(sim.pieces())
    runs = np.array(runs)
    for i in range(3):
        assert np.array_equal(gpu.pieces(i), runs[i])
    c = O.make_config(**kws[0])
    mask = O.mask_rule(c)
    orows, ojoin = EN.ensemble(c, mask, runs, R=24, seed=77)
    grows, gjoin = gpu.ensemble([0, 1, 2], R=24, seed=77)
    assert np.array_equal(gjoin, ojoin)
    ok = mask > 0
    assert np.array_equal(np.isfinite(grows), np.broadcast_to(ok, grows.shape))
    assert np.max(np.abs(grows[:, ok] - orows[:, ok])) < 1e-9
    # one run: every row is that run's concatenation
    one, _ = gpu.ensemble([2], R=3, seed=5)
    ref, _ = gpu.concat(2)
    for r in range(4):
        assert np.max(np.abs(one[r][ok] - ref[ok])) < 1e-12
    # order of runs is the draw order of resample 0
    rev, _ = gpu.ensemble([2, 1, 0], R=0, seed=1)
    orev, _ = EN.ensemble(c, mask, runs[::-1], R=0, seed=1)
    assert np.max(np.abs(rev[0][ok] - orev[0][ok])) < 1e-9
    with pytest.raises(rw.RewlError):
        gpu.ensemble([0, 5], R=1)
    gpu.close()


def test_ensemble_rejects_mismatched_runs(rw):
    a = dict(model="ising", L=8, n_windows=4, m=1, kfinal=8, X=100, seed=1)
    b = dict(a, L=10)
    gpu = rw.Rewl([rw.make_config(**a), rw.make_config(**b)])
    with pytest.raises(rw.RewlError):
        gpu.ensemble([0, 1], R=1)
    gpu.close()


def test_ensemble_full_size_potts_L100(rw):
    """The paper's smallest Potts lattice (q=10, L=100, 77 windows of 1001 bins,
    overlap 3/4): three runs whose window tables are set from known global tables
    (smooth + per-bin noise + per-run constant), mean + 6 resamples, then the
    canonical averages of every row."""
    from paper_1407_5140_amd import workloads as Wl
    base = dict(Wl.single("potts100"))
    base["m"] = 1
    kws = [dict(base, seed=s) for s in (1, 2, 3)]
    c = O.make_config(**kws[0])
    W = O.n_bins(c)
    lo, hi = O.layout(c)
    WB = int((hi - lo).max()) + 1
    rng = np.random.default_rng(100)
    b = np.arange(W)
    tables = []
    for j in range(3):
        t = 3000.0 * np.sin(np.pi * b / (W - 1)) + rng.normal(0, 0.02, W) + 17.0 * j
        tables.append(np.round(t * 2.0 ** 20) / 2.0 ** 20)
    gpu = rw.Rewl([rw.make_config(**kw) for kw in kws])
    for j in range(3):
        gpu.set_initial_lng(tables[j], j)
    runs = np.zeros((3, len(lo), WB))
    for j in range(3):
        for a in range(len(lo)):
            runs[j, a, : hi[a] - lo[a] + 1] = tables[j][lo[a]: hi[a] + 1]
    mask = O.mask_rule(c)
    orows, ojoin = EN.ensemble(c, mask, runs, R=6, seed=2024)
    grows, gjoin = gpu.ensemble([0, 1, 2], R=6, seed=2024)
    gpu.close()
    assert np.array_equal(gjoin, ojoin)
    ok = mask > 0
    assert np.max(np.abs(grows[:, ok] - orows[:, ok])) < 1e-9
    assert np.all(np.isneginf(grows[:, ~ok]))
    T = np.linspace(0.5, 3.0, 40)
    g = rw.rewl_thermo("potts", 100, orows, T)
    _assert_thermo(g, _oracle_thermo("potts", 100, orows, T))


# Shapes at the edges of the tiles (16 rows, 16 temperatures, blocks of 64 levels, 8 waves),
# grids narrow enough for the matrix path, wide ones, and one in no order.  Bounds as above.
@pytest.mark.parametrize("rows,temps", [(1, 1), (2, 7), (15, 8), (16, 9), (17, 16), (33, 17), (5, 33)])
@pytest.mark.parametrize("model,L", [("ising", 4), ("ising", 8), ("potts", 7), ("ising", 48), ("potts", 20)])
def test_thermo_shapes(rw, model, L, rows, temps):
    W = L * L + 1 if model == "ising" else 2 * L * L + 1
    rng = np.random.default_rng(rows * 100 + temps)
    x = np.linspace(-1, 1, W)
    lg = L * L * 0.69 * (1 - x ** 2) + rng.normal(0, 0.3, (rows, W))
    lg[:, rng.random(W) < 0.1] = -np.inf
    if W > 400:
        lg[0, 64:200] = -np.inf                                       # a whole block of absent levels
    lg[-1, :-1] = -np.inf                                             # one level: u exact, c = 0
    lg[-1, -1] = 1.0
    for T in (np.linspace(1.9, 2.1, temps), np.geomspace(0.1, 50.0, temps), rng.permutation(np.linspace(0.7, 3.0, temps))):
        _assert_thermo(rw.rewl_thermo(model, L, lg, T), _oracle_thermo(model, L, list(lg), T))


# The same on both sides of the 10 000 rows x temperatures from which the contraction is
# used: part tiles of rows, of temperatures and of 8 in 16, one temperature, many waves.
@pytest.mark.parametrize("rows,temps", [(99, 101), (100, 100), (17, 589), (10001, 1), (313, 33), (1, 10007)])
@pytest.mark.parametrize("model,L", [("ising", 4), ("potts", 7), ("ising", 33)])
def test_thermo_tiles(rw, model, L, rows, temps):
    W = L * L + 1 if model == "ising" else 2 * L * L + 1
    rng = np.random.default_rng(rows + temps)
    x = np.linspace(-1, 1, W)
    lg = L * L * 0.69 * (1 - x ** 2) + rng.normal(0, 0.3, (rows, W))
    lg[:, rng.random(W) < 0.1] = -np.inf
    lg[-1, :-1] = -np.inf
    lg[-1, -1] = 1.0
    some = sorted({0, rows // 2, rows - 2, rows - 1} - {-1})
    for T in (np.linspace(1.9, 2.1, temps), np.geomspace(0.1, 50.0, temps), rng.permutation(np.linspace(0.7, 3.0, temps))):
        g = rw.rewl_thermo(model, L, lg, T)
        _assert_thermo(tuple(np.asarray(x)[some] for x in g), _oracle_thermo(model, L, [lg[i] for i in some], T))


def test_thermo_names_the_first_bad_row(rw):
    lg = np.zeros((40, 65))
    for T in (np.linspace(2.0, 2.1, 20), np.geomspace(0.01, 50.0, 20)):
        for value, what in ((np.nan, "row 17: ln g holds NaN or"), (np.inf, "row 17: ln g holds NaN or"), (-np.inf, "row 17: no energy level")):
            bad = lg.copy()
            bad[30, 3] = np.nan
            if value == -np.inf:
                bad[17] = value
            else:
                bad[17, 64] = value
            with pytest.raises(rw.RewlError, match=what):
                rw.rewl_thermo("ising", 8, bad, T)


@pytest.mark.parametrize("L,h,overlap", [(16, 2, (3, 4)), (16, 3, (1, 10)), (24, 9, (9, 10)), (32, 64, (7, 8)),
                                         (32, 65, (9, 10)), (32, 66, (19, 20)), (40, 131, (29, 30))])
def test_ensemble_joins_of_many_overlaps(rw, L, h, overlap):
    """Overlaps many windows deep, so that a window's join often lies above where the next
    one was found on its own; more windows than the lanes of a wave.  Joins exact."""
    kws = [dict(model="ising", L=L, n_windows=h, overlap=overlap, m=1, kfinal=12, X=100, seed=s) for s in (1, 2, 3)]
    c = O.make_config(**kws[0])
    W, (lo, hi), mask = O.n_bins(c), O.layout(c), O.mask_rule(c)
    rng = np.random.default_rng(h)
    gpu = rw.Rewl([rw.make_config(**kw) for kw in kws])
    runs = np.zeros((3, h, int((hi - lo).max()) + 1))
    for j in range(3):
        t = np.round((L * np.sin(np.pi * np.arange(W) / W) + rng.normal(0, 0.1, W)) * 2.0 ** 16) / 2.0 ** 16
        gpu.set_initial_lng(t, j)
        for a in range(h):
            runs[j, a, : hi[a] - lo[a] + 1] = t[lo[a]: hi[a] + 1]
    grows, gjoin = gpu.ensemble([0, 1, 2], R=12, seed=9)
    gpu.close()
    orows, ojoin = EN.ensemble(c, mask, runs, R=12, seed=9)
    assert np.array_equal(gjoin, ojoin)
    ok = mask > 0
    assert np.max(np.abs(grows[:, ok] - orows[:, ok])) < 1e-9


@pytest.mark.parametrize("R", [255, 256, 1023, 1024, 2047, 2048])
@pytest.mark.parametrize("L,h", [(8, 1), (16, 9), (24, 33)])
def test_ensemble_of_many_rows(rw, L, h, R):
    """On both sides of the rows per CU at which the joining's blocks get smaller (256 CUs).
    Joins exact, of the first rows and of the last."""
    kws = [dict(model="ising", L=L, n_windows=h, overlap=(9, 10), m=1, kfinal=12, X=100, seed=s) for s in (1, 2)]
    c = O.make_config(**kws[0])
    W, (lo, hi), mask = O.n_bins(c), O.layout(c), O.mask_rule(c)
    rng = np.random.default_rng(h + R)
    gpu = rw.Rewl([rw.make_config(**kw) for kw in kws])
    runs = np.zeros((2, h, int((hi - lo).max()) + 1))
    for j in range(2):
        t = np.round((L * np.sin(np.pi * np.arange(W) / W) + rng.normal(0, 0.1, W)) * 2.0 ** 16) / 2.0 ** 16
        gpu.set_initial_lng(t, j)
        for a in range(h):
            runs[j, a, : hi[a] - lo[a] + 1] = t[lo[a]: hi[a] + 1]
    grows, gjoin = gpu.ensemble([0, 1], R=R, seed=9)
    gpu.close()
    orows, ojoin = EN.ensemble(c, mask, runs, R=24, seed=9)
    ok = mask > 0
    assert np.array_equal(gjoin[:25], ojoin) and np.max(np.abs(grows[:25][:, ok] - orows[:, ok])) < 1e-9
    last = EN.boot_picks(9, R, h, 2)[R]
    olast, jlast = EN.concat(c, mask, EN.mean_pieces(runs, last))
    assert np.array_equal(gjoin[R], jlast) and np.max(np.abs(grows[R][ok] - olast[ok])) < 1e-9


def test_ensemble_reports_an_overlap_without_a_join(rw):
    # overlaps of one bin: no five-point stencil fits
    kw = dict(model="ising", L=8, n_windows=4, overlap=(0, 1), m=1, kfinal=8, X=100)
    gpu = rw.Rewl([rw.make_config(seed=s, **kw) for s in (1, 2)])
    with pytest.raises(rw.RewlError, match="row 0: no valid join"):
        gpu.ensemble([0, 1], R=2)
    with pytest.raises(rw.RewlError, match="no valid join"):
        gpu.concat(1)
    gpu.close()


@pytest.mark.parametrize("rows,temps", [(8, 2000), (8, 1999), (7, 2287), (9, 1801), (17, 941), (33, 489), (16000, 1), (2003, 8)])
@pytest.mark.parametrize("model,L", [("ising", 4), ("potts", 7), ("ising", 33)])
def test_thermo_tiles_of_few_rows(rw, model, L, rows, temps):
    """As test_thermo_tiles, on both sides of 8 rows and of 16 000 rows x temperatures; low
    temperatures too, where one level has nearly all the weight."""
    W = L * L + 1 if model == "ising" else 2 * L * L + 1
    rng = np.random.default_rng(rows + temps)
    x = np.linspace(-1, 1, W)
    lg = L * L * 0.69 * (1 - x ** 2) + rng.normal(0, 0.3, (rows, W))
    lg[:, rng.random(W) < 0.1] = -np.inf
    lg[-1, :-1] = -np.inf
    lg[-1, -1] = 1.0
    some = sorted({0, rows // 2, rows - 2, rows - 1})
    for T in (np.linspace(1.9, 2.1, temps), np.geomspace(0.1, 50.0, temps), np.linspace(0.4, 0.44, temps)):
        g = rw.rewl_thermo(model, L, lg, T)
        _assert_thermo(tuple(np.asarray(x)[some] for x in g), _oracle_thermo(model, L, [lg[i] for i in some], T))


def test_thermo_takes_2_to_the_27_temperatures(rw):
    """32 threads to a temperature would be more than a launch can have; u alone, 1 GiB."""
    import ctypes
    lg, n = np.log(np.array([2.0, 1.0, 12.0, 1.0, 2.0])), (1 << 27) + 9
    T, u = np.full(n, 2.5), np.empty(n)
    T[-9:] = np.linspace(1.0, 3.0, 9)
    ref = rw.rewl_thermo("ising", 2, lg, T[-10:])[0][0]
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    assert rw._lib.rewl_thermo(0, 2, p(lg), 1, p(T), n, p(u), None, None) == rw.REWL_OK
    assert np.allclose(u[-10:], ref, rtol=1e-12, atol=0) and np.allclose(u[: n - 9: 1 << 20], ref[0], rtol=1e-12, atol=0)
