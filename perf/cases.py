"""The work that a program has this framework do, as cases that can be timed.

Four kinds, each through the package's public calls:

* ``call``      one exchange interval and the whole state, the way a small system is followed step
                by step (launch latency and the host path count as much as the chain).
* ``segment``   a stretch of exchange intervals of a run, its counters and its checkpoint: how long
                runs are driven (poll, look at the counters, save).  One instance or the batch.
* ``ensemble``  the n-run mean and its bootstrap resamples, joined into ln g over all bins.
* ``thermo``    canonical averages of many densities of states over a temperature grid.
* ``fit``, ``grad``, ``infer``  the density-of-states network: a stretch of training, one loss and
                gradient, and the evaluation over all levels of a target lattice.

Sizes are those of ``paper_1407_5140_amd.workloads``, of the ensemble study and of the warm start.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1407_5140_amd as rw
from paper_1407_5140_amd import workloads


# ------------------------------------------------------------------- cases
def _run(name, kind, model, q, L, h, m, X, n, **more):
    c = dict(kind=kind, model=model, q=q, L=L, h=h, m=m, X=X, intervals=n, pre=10, flat_num=4, flat_den=5,
             flat_rule="mean", exchange=True, tilted=False, graph=False, k0=0)
    c.update(more)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest lattice, one walker in each of four windows, looked at after every short interval;
        # the tight flatness keeps it from converging, after which a call would do nothing
        _run("ising8_call", "call", "ising", 2, 8, 4, 1, 1000, 1, flat_num=19, flat_den=20),
        # 128 walkers: far fewer chains than the GPU has SIMDs
        _run("ising32_segment", "segment", "ising", 2, 32, 8, 16, 10000, 20),
        # the benchmark's workload, 1 024 walkers, replayed as a graph
        _run("ising64_segment", "segment", "ising", 2, 64, 16, 64, 10000, 50, graph=True),
        # the ten-state Potts workload, 4 096 walkers
        _run("potts32_segment", "segment", "potts", 10, 32, 32, 128, 10000, 40),
        # the large Ising target: rows of two words, 2 048 walkers, narrow end windows
        _run("ising128_segment", "segment", "ising", 2, 128, 32, 64, 10000, 50, tilted=True),
        # the large Potts target: 4 096 walkers, counts that do not fit on chip
        _run("potts64_segment", "segment", "potts", 10, 64, 32, 128, 10000, 40, tilted=True),
        # 64 unequal instances in one handle, 65 280 walkers, with the tuning that the autotuner picks for it
        dict(name="batch64_segment", kind="batch", instances=64, X=10000, intervals=16, pre=2, sweep="lane",
             persistent=1, lds_kb=53, graph=True),
        # the error analysis of the L = 100 Potts study: four runs, 200 resamples, 77 windows
        dict(name="ensemble_potts100", kind="ensemble", model="potts", q=10, L=100, h=77, runs=4, R=200),
        # and its specific heat: 201 densities of states, 601 temperatures about the transition
        dict(name="thermo_potts100", kind="thermo", model="potts", q=10, L=100, rows=201, temps=601, T0=0.68, T1=0.74),
        # the warm start's network: a stretch of training, one gradient of a ragged batch, and the
        # table of every level of the Ising L = 128 target (16 385 rows, in chunks of the largest batch)
        dict(name="mlp_fit", kind="fit", in_dim=3, hidden=256, layers=3, max_batch=4096, rows=15265, batch=4096, steps=20),
        dict(name="mlp_grad_ragged", kind="grad", in_dim=3, hidden=256, layers=3, max_batch=4096, batch=1001),
        dict(name="mlp_infer_table", kind="infer", in_dim=3, hidden=256, layers=3, max_batch=4096, batch=16385),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["segment"] * 5 + ["call", "batch", "ensemble", "thermo", "fit", "grad", "infer"])
    if kind in ("segment", "call"):
        model = rng.choice(["ising", "potts"])
        small = kind == "call"
        if model == "ising":
            L, q = 2 * _log(rng, 4, 8 if small else 64), 2
        else:
            L, q = _log(rng, 8, 12 if small else 100), rng.randint(3, 16)
        W = L * L + 1 if model == "ising" else 2 * L * L + 1
        least = max(2, math.ceil(4 * W / 2000) - 3)     # windows of at most about 2 000 bins
        h = max(least, _log(rng, 2, max(3, min(90, W // 12))))
        m = 2 ** rng.randint(0, 2 if small else 7)
        while h * m > 4096 and m > 1:
            m //= 2
        X = _log(rng, 300, 3000) if small else _log(rng, 1000, 10000)
        n = 1 if small else max(1, min(100, int(1e6 * min(1.0, 1024 / (h * m)) * rng.uniform(0.3, 1.0) / X)))
        tight = L <= 16
        return _run(None, kind, model, q, L, h, m, X, n, flat_num=19 if tight else 4, flat_den=20 if tight else 5,
                    flat_rule=rng.choice(["mean", "mean", "visits"]) if not tight else "mean",
                    exchange=rng.random() < 0.85, tilted=h > 2 and rng.random() < 0.4, graph=rng.random() < 0.4)
    if kind == "batch":
        lane = rng.random() < 0.6
        return dict(kind="batch", instances=_log(rng, 4, 48), X=_log(rng, 1000, 10000), intervals=rng.randint(2, 16),
                    pre=2, sweep="lane" if lane else "auto", persistent=rng.randint(0, 1) if lane else 0,
                    lds_kb=rng.choice([0, 40, 53, 80]) if lane else 0, graph=rng.random() < 0.5)
    if kind == "ensemble":
        model = rng.choice(["ising", "potts"])
        L = 2 * _log(rng, 8, 50) if model == "ising" else _log(rng, 16, 100)
        W = L * L + 1 if model == "ising" else 2 * L * L + 1
        return dict(kind="ensemble", model=model, q=2 if model == "ising" else rng.randint(3, 12), L=L,
                    h=max(3, min(77, W // 60)), runs=rng.randint(2, 6), R=_log(rng, 20, 200))
    if kind == "thermo":
        model = rng.choice(["ising", "potts"])
        L = 2 * _log(rng, 8, 50) if model == "ising" else _log(rng, 16, 100)
        T0 = rng.uniform(1.5, 2.2) if model == "ising" else rng.uniform(0.6, 0.7)
        return dict(kind="thermo", model=model, q=2 if model == "ising" else rng.randint(3, 12), L=L,
                    rows=_log(rng, 1, 200), temps=_log(rng, 20, 600), T0=round(T0, 4), T1=round(T0 + rng.uniform(0.05, 0.5), 4))
    hidden, layers, most = 64 * rng.choice([1, 2, 3, 4, 4, 6, 8]), rng.randint(1, 5), 64 * rng.randint(8, 96)
    c = dict(kind=kind, in_dim=3, hidden=hidden, layers=layers, max_batch=most)
    if kind == "fit":
        return dict(c, rows=_log(rng, 500, 16000), batch=64 * rng.randint(1, most // 64), steps=rng.randint(5, 20))
    return dict(c, batch=rng.randint(1, most) if kind == "grad" else _log(rng, 1, 16000))


# ------------------------------------------------------------------ inputs
def _bins(c):
    N = c["L"] * c["L"]
    return N + 1 if c["model"] == "ising" else 2 * N + 1


def _levels(c):
    """E of every bin, and the bins whose level occurs."""
    N, W = c["L"] * c["L"], _bins(c)
    b = np.arange(W)
    ok = np.ones(W, bool)
    if c["model"] == "ising":
        ok[[1, N - 1]] = False
        return 4.0 * b - 2.0 * N, ok
    ok[[1, 2, 3, 5]] = False
    return b - 2.0 * N, ok


def _lng(c, seed, rows, rough):
    """Densities of states as runs find them: a concave ln g with a rough error of its own in each row."""
    rng = np.random.default_rng([seed, 77])
    E, ok = _levels(c)
    N = c["L"] * c["L"]
    u, top = E / N, math.log(2.0 if c["model"] == "ising" else c["q"])
    peak = 0.0 if c["model"] == "ising" else -2.0 / c["q"]
    s = top * (1.0 - ((u - peak) / (2.0 + peak)) ** 2)
    out = N * s[None, :] + rough * np.cumsum(rng.standard_normal((rows, len(E))), axis=1) / 8 + rough * rng.standard_normal((rows, len(E)))
    return out, ok


def _net_inputs(c, seed):
    """Flat parameters as the network starts with (uniform, 1/sqrt(fan in)), rows as the warm start encodes them."""
    rng = np.random.default_rng([seed, 5])
    H, parts, fan = c["hidden"], [], c["in_dim"]
    for _ in range(c["layers"]):
        parts += [rng.uniform(-1, 1, fan * H) / math.sqrt(fan), rng.uniform(-0.1, 0.1, H)]
        fan = H
    parts += [rng.uniform(-1, 1, H) / math.sqrt(H), rng.uniform(-0.1, 0.1, 1)]
    n = c["rows"] if c["kind"] == "fit" else c["batch"]
    q = rng.choice([2.0, 4.0, 8.0, 10.0], n)
    u = np.where(q == 2.0, rng.uniform(-2, 2, n), rng.uniform(-2, 0, n))
    x = np.stack([u, 1.0 / rng.integers(16, 129, n), q], axis=1).astype(np.float32)
    peak = np.where(q == 2.0, 0.0, -2.0 / q)
    t = np.log(q) * (1.0 - ((u - peak) / (2.0 + peak)) ** 2) + 0.01 * rng.standard_normal(n)
    return np.concatenate(parts).astype(np.float32), x, t.astype(np.float32)


def _config(c, seed, **more):
    kw = dict(model=c["model"], q=c["q"], L=c["L"], n_windows=c["h"], m=c["m"], X=c["X"], k0=c["k0"], kfinal=40,
              flat=(c["flat_num"], c["flat_den"]), flat_rule=c["flat_rule"], exchange=c["exchange"], seed=seed)
    kw.update(more)
    cfg = rw.make_config(**kw)
    return rw.make_config(windows=rw.tilted_layout(cfg), **kw) if c["tilted"] else cfg


def prepare(case, seed):
    c = case
    if c["kind"] in ("segment", "call"):
        g = rw.Rewl([_config(c, seed)], tune=rw.make_tune(use_graph=int(c["graph"]), poll_every=50))
        g.run(c["pre"])                                  # a run under way, off the start configurations
        return dict(case=c, g=g)
    if c["kind"] == "batch":
        cfgs = [rw.make_config(**dict(kw, seed=seed + i)) for i, kw in enumerate(workloads.batch(c["instances"], c["X"]))]
        g = rw.Rewl(cfgs, tune=rw.make_tune(kind=c["sweep"], persistent=c["persistent"], lds_target_kb=c["lds_kb"],
                                            use_graph=int(c["graph"]), poll_every=50))
        g.run(c["pre"])
        return dict(case=c, g=g)
    if c["kind"] == "ensemble":
        cfgs = [rw.make_config(model=c["model"], q=c["q"], L=c["L"], n_windows=c["h"], m=1, kfinal=20, seed=seed + i)
                for i in range(c["runs"])]
        g = rw.Rewl(cfgs)
        tab, _ = _lng(c, seed, c["runs"], 0.05)
        for i in range(c["runs"]):                       # each run's result, as its windows' tables hold it
            g.set_initial_lng(np.rint(tab[i] * 65536) / 65536, i)
        return dict(case=c, g=g, seed=seed)
    if c["kind"] == "thermo":
        lng, ok = _lng(c, seed, c["rows"], 0.05)
        lng[:, ~ok] = -np.inf
        return dict(case=c, lng=lng, T=np.linspace(c["T0"], c["T1"], c["temps"]))
    p, x, t = _net_inputs(c, seed)
    net = rw.Mlp(c["in_dim"], c["hidden"], c["layers"], max_batch=c["max_batch"], seed=1)
    net.set_params(p)
    return dict(case=c, net=net, x=x, t=t, seed=seed)


# --------------------------------------------------------------- one pass
_COUNTERS = ("intervals", "attempts", "windows_done", "min_k", "ex_prop", "ex_acc", "k", "round_trips", "slow_decisions")


def _counters(g, i):
    st = g.stats(i)
    return {key: st[key] for key in _COUNTERS}


def run(state):
    c = state["case"]
    if c["kind"] == "call":
        g = state["g"]
        g.run(c["intervals"])
        return g.state()
    if c["kind"] in ("segment", "batch"):
        g = state["g"]
        g.run(c["intervals"])
        counters = [_counters(g, i) for i in range(len(g.cfgs))]
        if len(counters) > 1:                            # one array per counter over all instances
            counters = {key: np.concatenate([np.atleast_1d(s[key]) for s in counters]) for key in _COUNTERS}
        return dict(counters=counters, checkpoint=np.frombuffer(rw.rewl_checkpoint(g.h), np.uint8))
    if c["kind"] == "ensemble":
        lng, join = state["g"].ensemble(range(c["runs"]), c["R"], state["seed"])
        return dict(lng=lng, join=join)
    if c["kind"] == "thermo":
        u, cv, f = rw.rewl_thermo(c["model"], c["L"], state["lng"], state["T"])
        return dict(u=u, c=cv, f=f)
    net = state["net"]
    if c["kind"] == "fit":
        loss = net.fit(state["x"], state["t"], c["steps"], batch=c["batch"], lr=1e-3, seed=state["seed"] & 0xffffffff)
        return dict(loss=np.float32(loss), params=net.params())
    if c["kind"] == "grad":
        g, loss = net.grad(state["x"], state["t"])
        return dict(grad=g, loss=np.float32(loss))
    return dict(y=net.infer(state["x"]))


# ------------------------------------------------------------------- work
def _state_bytes(kw):
    L, h, m = kw["L"], kw["h"], kw["m"]
    N = L * L
    W = N + 1 if kw["model"] == "ising" else 2 * N + 1
    WB = math.ceil((W - 1) * 4 / (h + 3)) + 1            # equal windows of 75 % overlap
    lattice = N / 8 if kw["model"] == "ising" else N
    return h * m * (lattice + 8 * WB + 16) + h * WB * 8


def work(case):
    """The walkers' state read and written once and the arithmetic of the attempts themselves
    (30 operations for an Ising attempt, 37 for a Potts one); for the others inputs and outputs once."""
    c = case
    if c["kind"] in ("segment", "call"):
        ops = 30 if c["model"] == "ising" else 37
        return dict(bytes=2 * _state_bytes(c), flops=float(ops) * c["X"] * c["h"] * c["m"] * c["intervals"])
    if c["kind"] == "batch":
        by = fl = 0.0
        for kw in workloads.batch(c["instances"], c["X"]):
            kw["h"] = kw["n_windows"]
            by += 2 * _state_bytes(kw)
            fl += (30 if kw["model"] == "ising" else 37) * float(c["X"]) * kw["h"] * kw["m"] * c["intervals"]
        return dict(bytes=by, flops=fl)
    if c["kind"] == "ensemble":
        W = _bins(c)
        WB = math.ceil((W - 1) * 4 / (c["h"] + 3)) + 1
        rows = c["R"] + 1
        return dict(bytes=8.0 * (c["runs"] * c["h"] * WB + rows * W), flops=float(rows) * c["h"] * WB * c["runs"])
    if c["kind"] == "thermo":
        W = _bins(c)
        return dict(bytes=8.0 * c["rows"] * (W + 3 * c["temps"]), flops=25.0 * c["rows"] * W * c["temps"])
    H, layers, B = c["hidden"], c["layers"], c["batch"]
    P = c["in_dim"] * H + H + (layers - 1) * (H * H + H) + H + 1
    forward = 2.0 * B * (c["in_dim"] * H + (layers - 1) * H * H + H)
    if c["kind"] == "fit":                               # parameters and both moments in and out, the rows in
        return dict(bytes=4.0 * (6 * P + c["rows"] * (c["in_dim"] + 1)), flops=3.0 * forward * c["steps"])
    if c["kind"] == "grad":
        return dict(bytes=4.0 * (2 * P + B * (c["in_dim"] + 1)), flops=3.0 * forward)
    return dict(bytes=4.0 * (P + B * (c["in_dim"] + 1)), flops=forward)


# ---------------------------------------------------------- 64-bit results
def _philox_x0(ctr, key):
    """First word of Philox4x32-10 (Salmon et al., SC'11) at counters ctr[4] (arrays) under a two-word key."""
    c0, c1, c2, c3 = (np.asarray(v, np.uint64) for v in ctr)
    k0, k1 = key
    low = np.uint64(0xffffffff)
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c0, np.uint64(0xCD9E8D57) * c2
        c0, c1, c2, c3 = ((p1 >> np.uint64(32)) ^ c1 ^ np.uint64(k0), p1 & low, (p0 >> np.uint64(32)) ^ c3 ^ np.uint64(k1), p0 & low)
        k0, k1 = (k0 + 0x9E3779B9) & 0xffffffff, (k1 + 0xBB67AE85) & 0xffffffff
    return c0


def _exact_ensemble(c, seed):
    tab, ok = _lng(c, seed, c["runs"], 0.05)
    tab = np.rint(tab * 65536) / 65536
    W, h, n, R = _bins(c), c["h"], c["runs"], c["R"]
    S = W - 1
    w = min(S, -(-S * 4 // (4 + (h - 1))))
    lo = [a * (S - w) // (h - 1) for a in range(h)]
    pieces = []
    r = np.arange(1, R + 1)
    for a in range(h):
        acc = np.zeros((R + 1, w + 1))
        for j in range(n):
            x0 = _philox_x0((r, np.full(R, j), np.full(R, a), np.full(R, 4)), (seed & 0xffffffff, seed >> 32))
            pick = np.concatenate([[j], (x0 * np.uint64(n)) >> np.uint64(32)]).astype(np.int64)
            acc += tab[pick, lo[a]:lo[a] + w + 1]
        pieces.append(acc / n)
    out = np.empty((R + 1, W))
    for s in range(R + 1):
        shift, first, out[s, : w + 1] = 0.0, 0, pieces[0][s]
        for a in range(h - 1):
            fa, fb, ov = pieces[a][s], pieces[a + 1][s], lo[a] + w - lo[a + 1] + 1
            d = min(10, max(1, ov // 8))
            b = np.arange(max(lo[a + 1] + 2 * d, first), lo[a] + w - 2 * d + 1)
            b = b[ok[b] & ok[b - d] & ok[b + d] & ok[b - 2 * d] & ok[b + 2 * d]]
            slope = [((f[b - o - 2 * d] - 8.0 * f[b - o - d]) + 8.0 * f[b - o + d]) - f[b - o + 2 * d] for f, o in ((fa, lo[a]), (fb, lo[a + 1]))]
            at = b[np.argmin(np.abs(slope[0] / (12.0 * d) - slope[1] / (12.0 * d)))]
            shift, first = shift + (fa[at - lo[a]] - fb[at - lo[a + 1]]), at + 1
            out[s, at + 1: lo[a + 1] + w + 1] = fb[at + 1 - lo[a + 1]:] + shift
    out[:, ~ok] = -np.inf
    top = out.max(axis=1, keepdims=True)
    norm = top + np.log(np.exp(out - top).sum(axis=1, keepdims=True))
    return out + (c["L"] ** 2 * math.log(2.0 if c["model"] == "ising" else c["q"]) - norm)


def _exact_thermo(c, seed):
    lng, ok = _lng(c, seed, c["rows"], 0.05)
    E = torch.from_numpy(_levels(c)[0][ok])
    g = torch.from_numpy(np.ascontiguousarray(lng[:, ok]))
    N = c["L"] ** 2
    T = torch.from_numpy(np.linspace(c["T0"], c["T1"], c["temps"]))
    u, cv, f = (torch.empty(c["rows"], c["temps"], dtype=torch.float64) for _ in range(3))
    for k in range(c["temps"]):
        x = g - E / T[k]
        top = x.max(dim=1, keepdim=True).values
        x -= top
        some = (x.max(dim=0).values > -746.0).nonzero()[:, 0]    # elsewhere every weight is zero in 64 bits
        at = slice(int(some[0]), int(some[-1]) + 1)
        p, e = torch.exp(x[:, at]), E[at]
        Z = p.sum(dim=1, keepdim=True)
        mean = (p @ e)[:, None] / Z
        var = (p * (e - mean) ** 2).sum(dim=1, keepdim=True) / Z
        u[:, k], cv[:, k] = mean[:, 0] / N, var[:, 0] / (N * T[k] ** 2)
        f[:, k] = (-T[k] * (top + torch.log(Z)) / N)[:, 0]
    return dict(u=u, c=cv, f=f)


def _exact_net(c, seed):
    """The network in 64 bits (with its gradient for ``grad``), from the 32-bit parameters and rows."""
    p, x, t = _net_inputs(c, seed)
    p = torch.from_numpy(p).double().requires_grad_(c["kind"] == "grad")
    a, fan, at, H = torch.from_numpy(x).double(), c["in_dim"], 0, c["hidden"]
    for _ in range(c["layers"]):
        W, b = p[at: at + fan * H].reshape(fan, H), p[at + fan * H: at + fan * H + H]
        at += fan * H + H
        a, fan = torch.nn.functional.gelu(a @ W + b), H
    y = a @ p[at: at + H] + p[at + H]
    if c["kind"] == "infer":
        return dict(y=y)
    loss = ((y - torch.from_numpy(t).double()) ** 2).mean()
    loss.backward()
    return dict(grad=p.grad, loss=loss.detach())


def exact(case, seed):
    c = case
    if c["kind"] == "ensemble":
        return dict(lng=_exact_ensemble(c, seed), join=None)
    if c["kind"] == "thermo":
        return _exact_thermo(c, seed)
    if c["kind"] in ("grad", "infer"):
        return _exact_net(c, seed)
    return None                                          # random walks, and training on drawn rows
