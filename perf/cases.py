"""The calls whose speed counts: what a program that uses libte has it do, by entry point and size.

A case names the call (``kind``) and its sizes; ``prepare`` makes what the program holds before the
call (series on the GPU, the plan, its workspace, the server), ``run`` makes the call once.  Series
are coupled autoregressive pairs or 1/f noise, drawn from the seed: the processes that the
repository's own workloads use, at those workloads' sizes or odd ones of the same ranges.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

import paper_1401_4068_amd as te


def listed():
    return [
        # one window of one pair, no surrogates: the smallest useful call, all latency
        dict(name="single_window", kind="surrogates", proc="linear", pairs=1, R=100, T=100, d_y=2, d_x=2, tau=1,
             u=1, k=4, points=1, W=20, S=0, perms="none"),
        # the plain per-window path over a few windows of odd size, as an exploratory script calls it
        dict(name="estimate_windows", kind="estimate", proc="linear", pairs=1, R=73, T=160, d_y=2, d_x=1, tau=2,
             u=3, k=4, points=6, W=17, S=0, perms="none"),
        # time-resolved ensemble estimate: many windows, all trials pooled, no surrogates
        dict(name="ensemble", kind="surrogates", proc="nonlinear", pairs=1, R=500, T=300, d_y=3, d_x=3, tau=1, u=3,
             k=4, points=100, W=10, S=0, perms="none"),
        # one long window alone: a large search space with few reference blocks
        dict(name="long_window", kind="surrogates", proc="linear", pairs=1, R=2400, T=60, d_y=3, d_x=3, tau=1, u=1,
             k=4, points=1, W=20, S=0, perms="none"),
        # windows of 1 000 to 50 000 points, each with its surrogates drawn by the library: the bench's batch, smaller
        dict(name="uneven_surrogates", kind="uneven", proc="linear", pairs=1, R=5000, T=400, d_y=3, d_x=3, tau=1,
             u=1, k=4, points=30, W=0, S=100, perms="none"),
        # many channel pairs, wide embedding, small windows, the caller's own permutations
        dict(name="channel_pairs", kind="surrogates", proc="pink", pairs=8, R=120, T=1200, d_y=4, d_x=4, tau=2, u=5,
             k=4, points=40, W=20, S=100, perms="given"),
        # delay reconstruction of both directions: every assumed delay, then surrogates at the best one
        dict(name="delay_scan", kind="delay_scan", proc="ar3", pairs=2, R=50, T=3000, d_y=2, d_x=1, tau=1, u=1, k=4,
             points=8, W=300, S=300, perms="none", n_u=30),
        # local transfer entropy of every pooled point
        dict(name="local_te", kind="local", proc="nonlinear", pairs=1, R=500, T=120, d_y=3, d_x=2, tau=1, u=3, k=4,
             points=5, W=21, S=0, perms="none"),
        # neighbour search over pre-embedded chunks of odd sizes, k other than 4
        dict(name="knn_counts", kind="knn", d_y=2, d_x=3, k=6, chunks=9, n_lo=801, n_hi=12007),
        # conditioning on the current source sample, surrogates with the caller's permutations
        dict(name="conditioned", kind="surrogates", proc="linear", pairs=1, R=61, T=240, d_y=2, d_x=2, tau=1, u=2,
             k=5, points=10, W=19, S=40, perms="given", cond=1),
        # choice of the target's embedding among twelve candidates, with the predictions
        dict(name="embedding_choice", kind="ragwitz", proc="ar1", R=50, T=3000, W=300, start=1100, k=4, d_max=6,
             tau_max=2),
        # a burst of jobs of mixed shapes through the server
        dict(name="served_jobs", kind="served", jobs=16, n_lo=1000, n_hi=20000, s_max=100),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "estimate", "ensemble", "long", "uneven", "pairs", "delay_scan", "local", "knn",
                       "cond", "ragwitz", "served"])
    k = rng.choice([4, 4, 4, 1, 3, 5, 8])
    dims = dict(d_y=rng.randint(1, 4), d_x=rng.randint(1, 4), tau=rng.randint(1, 2), u=rng.randint(1, 5))
    if kind == "small":
        return dict(kind="surrogates", proc=rng.choice(["linear", "nonlinear"]), pairs=1, R=_log(rng, 20, 400), T=90,
                    k=k, points=rng.randint(1, 4), W=rng.randint(5, 25), S=0, perms="none", **dims)
    if kind == "estimate":
        return dict(kind="estimate", proc="linear", pairs=1, R=_log(rng, 40, 900), T=150, k=k,
                    points=rng.randint(2, 9), W=rng.randint(9, 25), S=0, perms="none", **dims)
    if kind == "ensemble":
        return dict(kind="surrogates", proc="nonlinear", pairs=1, R=_log(rng, 100, 700), T=300, k=k,
                    points=rng.randint(40, 120), W=rng.randint(7, 14), S=0, perms="none", **dims)
    if kind == "long":
        return dict(kind="surrogates", proc="linear", pairs=1, R=_log(rng, 600, 3000), T=70, k=4, points=1,
                    W=rng.randint(11, 25), S=0, perms="none", **dims)
    if kind == "uneven":
        d = rng.randint(2, 4)
        return dict(kind="uneven", proc="linear", pairs=1, R=rng.randint(1000, 3000), T=200, d_y=d, d_x=d, tau=1,
                    u=1, k=4, points=rng.randint(6, 16), W=0, S=rng.randint(20, 60), perms="none")
    if kind == "pairs":
        return dict(kind="surrogates", proc="pink", pairs=rng.randint(2, 6), R=rng.randint(60, 150), T=600, k=4,
                    points=rng.randint(8, 30), W=rng.randint(9, 24), S=rng.randint(20, 100),
                    perms=rng.choice(["none", "given"]), **dims)
    if kind == "delay_scan":
        return dict(kind="delay_scan", proc="ar1", pairs=2, R=rng.randint(20, 50), T=1500, d_y=rng.randint(1, 3),
                    d_x=rng.randint(1, 2), tau=1, u=1, k=4, points=rng.randint(1, 4), W=rng.randint(101, 300),
                    S=rng.randint(0, 200), perms="none", n_u=rng.randint(5, 20))
    if kind == "local":
        return dict(kind="local", proc="nonlinear", pairs=1, R=_log(rng, 80, 800), T=150, k=k,
                    points=rng.randint(1, 8), W=rng.randint(10, 30), S=0, perms="none", **dims)
    if kind == "knn":
        lo = _log(rng, 100, 3000)
        return dict(kind="knn", d_y=dims["d_y"], d_x=dims["d_x"], k=rng.randint(1, 15), chunks=rng.randint(1, 20),
                    n_lo=lo, n_hi=lo * rng.randint(2, 6))
    if kind == "cond":
        return dict(kind="surrogates", proc="linear", pairs=rng.randint(1, 2), R=_log(rng, 30, 300), T=200,
                    d_y=rng.randint(1, 3), d_x=dims["d_x"], tau=1, u=dims["u"], k=k, points=rng.randint(2, 12),
                    W=rng.randint(8, 22), S=rng.randint(10, 60), perms=rng.choice(["none", "given"]), cond=1)
    if kind == "ragwitz":
        return dict(kind="ragwitz", proc="ar1", R=rng.randint(10, 50), T=2000, W=rng.randint(51, 300), start=1100,
                    k=k, d_max=rng.randint(2, 8), tau_max=rng.randint(1, 2))
    return dict(kind="served", jobs=rng.randint(4, 20), n_lo=600, n_hi=rng.randint(4000, 16000),
                s_max=rng.randint(20, 100))


# ---------------------------------------------------------------------------- series

def _ar_pair(rng, R, T, delay, nonlinear):
    """x_t = 0.5 x_{t-1} + e,  y_t = 0.5 y_{t-1} + c f(x_{t-delay}) + e'."""
    n = T + 60
    ex, ey = rng.standard_normal((2, n, R))
    x, y = np.zeros((n, R)), np.zeros((n, R))
    for t in range(1, n):
        x[t] = 0.5 * x[t - 1] + ex[t]
        drive = x[t - delay] if t >= delay else 0.0
        y[t] = 0.5 * y[t - 1] + (0.3 * np.tanh(drive) if nonlinear else 0.4 * drive) + ey[t]
    return x[60:].T, y[60:].T


def _scenario(rng, R, T, both):
    """Two AR(1) processes whose coupling sets in at sample 1000 (and the other direction at 2000)."""
    n = T + 60
    t = np.arange(n) - 60.0
    gxy = -0.35 * 0.5 * (1 + np.tanh(0.05 * (t - 1000)))
    gyx = -0.4 * 0.5 * (1 + np.tanh(0.05 * (t - 2000))) * (1.0 if both else 0.0)
    ex, ey = rng.standard_normal((2, n, R))
    x, y = np.zeros((n, R)), np.zeros((n, R))
    ax = 0.475 if both else 0.75
    for i in range(1, n):
        x[i] = ax * x[i - 1] + (gyx[i] * y[i - 20] if i >= 20 else 0.0) + ex[i]
        y[i] = 0.35 * y[i - 1] + (gxy[i] * x[i - 10] if i >= 10 else 0.0) + ey[i]
    return x[60:].T, y[60:].T


def _pink(rng, R, T):
    f = np.fft.rfftfreq(T)
    g = np.zeros_like(f)
    g[1:] = f[1:] ** -0.5
    s = np.fft.irfft(np.fft.rfft(rng.standard_normal((R, T)), axis=1) * g, n=T, axis=1)
    return (s - s.mean(axis=1, keepdims=True)) / s.std(axis=1, keepdims=True)


def _series(c, rng):
    R, T, proc = c["R"], c["T"], c["proc"]
    xs, ys = [], []
    for _ in range(c["pairs"]):
        if proc in ("ar1", "ar3"):
            a, b = _scenario(rng, R, T, proc == "ar3")
            xs, ys = [a, b][: c["pairs"]], [b, a][: c["pairs"]]      # both directions as two pairs
            break
        if proc == "pink":
            a, b = _pink(rng, R, T), _pink(rng, R, T)
            b[:, 5:] += 0.4 * a[:, :-5] * (np.arange(5, T) < T // 2)
        else:
            a, b = _ar_pair(rng, R, T, max(1, c["u"]), proc == "nonlinear")
        xs.append(a)
        ys.append(b)
    return np.stack(xs).astype(np.float32, order="C"), np.stack(ys).astype(np.float32, order="C")


def _geometry(c):
    """Window starts, lengths and pooled trials: fixed by the case."""
    h = max(1 + (c["d_y"] - 1) * c["tau"], (c.get("n_u") or c["u"]) + (c["d_x"] - 1) * c["tau"])
    C, R, T = c["points"], c["R"], c["T"]
    if c["kind"] == "uneven":
        g = np.random.default_rng(C * 7919 + R)
        W = g.integers(10, 21, C)
        trials = np.clip(np.rint(g.uniform(1000, min(50000, 10 * R), C) / W), 50, R).astype(np.int32)
    else:
        W, trials = np.full(C, c["W"]), np.full(C, R, np.int32)
    start = h + (np.arange(C) * max(0, T - int(W.max()) - h)) // max(C - 1, 1)
    if c["kind"] == "delay_scan":
        start = 200 + np.arange(C) * ((T - 200 - c["W"]) // max(C - 1, 1) if C > 1 else 0)
    return start.astype(np.int32), W.astype(np.int32), trials


def _perms(c, rng):
    """int32 [pairs, points, S, R], uniform trial permutations."""
    n = c["pairs"] * c["points"] * c["S"]
    p = np.argsort(rng.random((n, c["R"]), dtype=np.float32), axis=1).astype(np.int32)
    return p.reshape(c["pairs"], c["points"], c["S"], c["R"])


def _knn_points(c, rng):
    sizes = np.round(np.exp(np.linspace(math.log(c["n_lo"]), math.log(c["n_hi"]), c["chunks"]))).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    y = rng.standard_normal((c["d_y"] + 1, n))
    x = rng.standard_normal((c["d_x"], n))
    for m in range(c["d_y"] - 1, -1, -1):
        y[m] += 0.5 * y[m + 1]                       # y_t | y_{t-1}, y_{t-2}, ...
    y[0] += 0.4 * x[0]
    return np.concatenate([y, x]).astype(np.float32), off


def _jobs(c, rng):
    jobs = []
    for j in range(c["jobs"]):
        d, W = int(rng.integers(2, 5)), int(rng.choice([10, 20]))
        n = math.exp(rng.uniform(math.log(c["n_lo"]), math.log(c["n_hi"])))
        R = max(8, int(round(n / W)))
        jobs.append(types.SimpleNamespace(
            x=None, y=None, n_pairs=1, n_trials=R, n_samples=d + W, d_y=d,
            d_x=d, tau=1, u=1, k=4, window_start=np.array([d], np.int32), window_len=np.array([W], np.int32),
            trials=np.array([R], np.int32), n_points=1, n_surrogates=int(rng.integers(0, c["s_max"] + 1)),
            perms=None, perm_seed=int(rng.integers(1 << 30)), cond_source=0))
    return jobs


def _inputs(c, seed):
    rng = np.random.default_rng([seed, 1401])
    if c["kind"] == "knn":
        return _knn_points(c, rng)
    if c["kind"] == "served":
        shape = np.random.default_rng([c["jobs"], c["n_hi"], c["s_max"]])     # shapes by the case, values by the seed
        jobs = _jobs(c, shape)
        for j in jobs:
            a, b = _ar_pair(rng, j.n_trials, j.n_samples, 1, False)
            j.x, j.y = a[None].astype(np.float32, order="C"), b[None].astype(np.float32, order="C")
        return jobs
    if c["kind"] == "ragwitz":
        x, y = _scenario(rng, c["R"], c["T"], False)
        return (y.astype(np.float32, order="C"),)
    x, y = _series(c, rng)
    perms = _perms(c, rng) if c["perms"] == "given" and c["S"] else None
    return x, y, perms


def _candidates(c):
    return [(d, t) for t in range(1, c["tau_max"] + 1) for d in range(1, c["d_max"] + 1)]


def prepare(case, seed):
    c = case
    s = types.SimpleNamespace(c=c)
    if c["kind"] == "served":
        s.jobs = _inputs(c, seed)
        s.server = te.Server(4 << 30)
        return s
    if c["kind"] == "knn":
        pts, s.off = _inputs(c, seed)
        s.pts = torch.from_numpy(pts).cuda()
        s.ws = torch.empty(te.lib().te_knn_counts_workspace_bytes(c["chunks"], int(s.off[-1])), dtype=torch.uint8,
                           device="cuda")
        return s
    if c["kind"] == "ragwitz":
        s.y = torch.from_numpy(_inputs(c, seed)[0]).cuda()
        return s
    x, y, perms = _inputs(c, seed)
    start, W, trials = _geometry(c)
    s.x, s.y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    s.perms = None if perms is None else torch.from_numpy(perms).cuda()
    s.plan = te.Plan(c["pairs"], c["R"], c["T"], c["d_y"], c["d_x"], c["tau"], c["u"], c["k"], start, W, trials,
                     c["S"], cond_source=c.get("cond", 0), seed=seed)
    if c["kind"] == "delay_scan":
        s.us = list(range(1, c["n_u"] + 1))
        s.ws = torch.empty(int(s.plan.delay_scan_workspace_bytes(s.us)[0]), dtype=torch.uint8, device="cuda")
    else:
        s.ws = s.plan.workspace()
    return s


def run(state):
    s = state
    kind = s.c["kind"]
    if kind in ("surrogates", "uneven"):
        return s.plan.surrogates(s.x, s.y, s.perms, ws=s.ws)
    if kind == "estimate":
        return s.plan.estimate(s.x, s.y, ws=s.ws)
    if kind == "local":
        return s.plan.local(s.x, s.y, ws=s.ws)
    if kind == "delay_scan":
        r = s.plan.delay_scan(s.x, s.y, s.us, s.perms, ws=s.ws)
        return [v for v in r if v is not None]
    if kind == "knn":
        return te.knn_counts(s.pts, s.off, s.c["d_y"], s.c["d_x"], s.c["k"], ws=s.ws)
    if kind == "ragwitz":
        return te.ragwitz(s.y, s.c["start"], s.c["W"], _candidates(s.c), s.c["k"], want_pred=True)
    tickets = [s.server.submit(j) for j in s.jobs]
    return [v for t in tickets for v in s.server.wait(t)]


# ------------------------------------------------------------------- what a pass cannot do without

def _search_ops(n, D, chunks):
    """Operations of a search that reaches every point's neighbours through an index, without a visit to
    the points outside: a descent of log2 n levels and 4D + 2 operations per level."""
    return chunks * n * math.log2(max(n, 2)) * (4 * D + 2)


def work(case):
    c = case
    if c["kind"] == "served":
        b = f = 0
        for j in _jobs(c, np.random.default_rng([c["jobs"], c["n_hi"], c["s_max"]])):
            n = j.n_trials * int(j.window_len[0])
            b += 8 * j.n_trials * j.n_samples + 8 * (j.n_surrogates + 2)
            f += _search_ops(n, 1 + 2 * j.d_y, 1 + j.n_surrogates)
        return {"bytes": b, "flops": f}
    if c["kind"] == "knn":
        off = _knn_sizes(c)
        D = 1 + c["d_y"] + c["d_x"]
        return {"bytes": int(off.sum()) * (4 * D + 16), "flops": sum(_search_ops(int(n), D, 1) for n in off)}
    if c["kind"] == "ragwitz":
        n, cand = c["R"] * c["W"], _candidates(c)
        span = c["W"] + 1 + (c["d_max"] - 1) * c["tau_max"]
        return {"bytes": 4 * c["R"] * span + 8 * n * len(cand), "flops": sum(_search_ops(n, d, 1) for d, _ in cand)}
    start, W, trials = _geometry(c)
    n = W.astype(np.int64) * trials
    D = 1 + c["d_y"] + c["d_x"] + c.get("cond", 0)
    chunks = 1 + c["S"] + c.get("n_u", 0)
    b = 8 * c["pairs"] * int((trials.astype(np.int64) * W).sum()) + 8 * c["pairs"] * c["points"] * (chunks + 1)
    if c["perms"] == "given":
        b += 4 * c["pairs"] * c["points"] * c["S"] * c["R"]
    if c["kind"] == "local":
        b += 8 * int(n.sum())
    return {"bytes": b, "flops": c["pairs"] * sum(_search_ops(int(v), D, chunks) for v in n)}


def _knn_sizes(c):
    return np.round(np.exp(np.linspace(math.log(c["n_lo"]), math.log(c["n_hi"]), c["chunks"]))).astype(np.int64)


# ------------------------------------------------------------------------------------ in 64 bits

def _psi(n):
    return torch.special.digamma(n.to(torch.float64))


def _ksg(p, d_y, d_x, k):
    """Radii, counts and per-point terms of one chunk: p float32 [D, n].  Distances are the interface's
    binary32 coordinate differences; everything summed is in 64 bits."""
    n = p.shape[1]
    eps = torch.empty(n, dtype=torch.float32, device=p.device)
    cnt = torch.empty((3, n), dtype=torch.int64, device=p.device)
    step = max(1, (1 << 26) // n)
    for a in range(0, n, step):
        b = min(n, a + step)
        i = torch.arange(b - a, device=p.device)

        def block(ms):
            d = None
            for m in ms:
                v = (p[m, a:b, None] - p[m][None, :]).abs_()
                d = v if d is None else torch.maximum(d, v, out=d)
            return d
        t, q, s = block([0]), block(range(1, 1 + d_y)), block(range(1 + d_y, 1 + d_y + d_x))
        j = torch.maximum(torch.maximum(t, q), s)
        j[i, a + i] = math.inf
        e = j.topk(k, dim=1, largest=False, sorted=True).values[:, -1]
        eps[a:b] = e
        e = e[:, None]
        for row, d in enumerate((q, torch.maximum(t, q), torch.maximum(q, s))):
            d[i, a + i] = math.inf
            cnt[row, a:b] = (d < e).sum(1)
    term = _psi(torch.tensor(k, device=p.device)) + _psi(cnt[0] + 1) - _psi(cnt[1] + 1) - _psi(cnt[2] + 1)
    return eps, cnt, term


def _embed(c, x, y, w, W, Rc, phi=None):
    t = torch.arange(w, w + W, device=x.device)
    src = x[:Rc] if phi is None else x[phi[:Rc].long()]
    rows = [y[:Rc][:, t]] + [y[:Rc][:, t - 1 - m * c["tau"]] for m in range(c["d_y"])]
    if c.get("cond"):
        rows.append(src[:, t])
    rows += [src[:, t - c["u"] - m * c["tau"]] for m in range(c["d_x"])]
    return torch.stack([r.reshape(-1) for r in rows]), c["d_y"] + c.get("cond", 0)


def _pairs(c):
    """Point pairs of a whole pass: what a brute-force value costs."""
    if c["kind"] == "knn":
        return int((_knn_sizes(c) ** 2).sum())
    if c["kind"] == "ragwitz":
        return (c["R"] * c["W"]) ** 2 * c["d_max"] * c["tau_max"]
    start, W, trials = _geometry(c)
    return int(((W.astype(np.int64) * trials) ** 2).sum()) * c["pairs"] * (1 + c["S"])


def exact(case, seed):
    c = case
    if c["kind"] in ("served", "uneven", "delay_scan") or _pairs(c) > 6e9:
        return None
    if c["kind"] == "knn":
        pts, off = _inputs(c, seed)
        p = torch.from_numpy(pts).cuda()
        got = [_ksg(p[:, off[i]:off[i + 1]].contiguous(), c["d_y"], c["d_x"], c["k"]) for i in range(c["chunks"])]
        return (torch.cat([g[0] for g in got]), torch.cat([g[1] for g in got], 1).to(torch.int32),
                np.array([float(g[2].mean()) for g in got]))
    if c["kind"] == "ragwitz":
        y = torch.from_numpy(_inputs(c, seed)[0]).cuda()
        t = torch.arange(c["start"], c["start"] + c["W"], device="cuda")
        tgt = y[:, t].reshape(-1).to(torch.float64)
        n = tgt.shape[0]
        scores, preds = [], []
        for d, tau in _candidates(c):
            p = torch.stack([y[:, t - 1 - m * tau].reshape(-1) for m in range(d)])
            pred = torch.empty(n, dtype=torch.float64, device="cuda")
            step = max(1, (1 << 25) // n)
            for a in range(0, n, step):
                b = min(n, a + step)
                i = torch.arange(b - a, device="cuda")
                dist = (p[0, a:b, None] - p[0][None, :]).abs_()
                for m in range(1, d):
                    torch.maximum(dist, (p[m, a:b, None] - p[m][None, :]).abs_(), out=dist)
                dist[i, a + i] = math.inf
                # equal distances rank by index: the distance's bits, then the index, in one integer
                key = (dist.view(torch.int32).to(torch.int64) << 32) | torch.arange(n, device="cuda")
                near = key.topk(c["k"], dim=1, largest=False, sorted=True).values & 0xFFFFFFFF
                pred[a:b] = tgt[near].sum(1) / c["k"]
            preds.append(pred)
            scores.append(float(((tgt - pred) ** 2).sum() / ((tgt - tgt.mean()) ** 2).sum()))
        return np.array(scores), torch.stack(preds)
    x, y, perms = _inputs(c, seed)
    if c["S"] and perms is None:
        return None                               # the library draws these permutations itself
    x, y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    start, W, trials = _geometry(c)
    est = np.empty((c["pairs"], c["points"], 1 + c["S"]))
    local = []
    for p in range(c["pairs"]):
        for w in range(c["points"]):
            for s in range(1 + c["S"]):
                phi = torch.from_numpy(perms[p, w, s - 1]).cuda() if s else None
                pts, d_p = _embed(c, x[p], y[p], int(start[w]), int(W[w]), int(trials[w]), phi)
                term = _ksg(pts, d_p, c["d_x"], c["k"])[2]
                est[p, w, s] = float(term.mean())
                local.append(term)
    if c["kind"] == "estimate":
        return est[:, :, 0]
    if c["kind"] == "local":
        return local, est[:, :, 0]
    # a p-value counts comparisons of estimates: a whole number over S, not a rounded one
    return est[:, :, 0], est[:, :, 1:], None
