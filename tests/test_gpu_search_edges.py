"""GPU tests of the searches where their inputs or launch shapes are unusual."""
import numpy as np
import pytest

import synth
from synth.rng import derive_key, normal64, stream_u64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def te():
    import paper_1401_4068_amd as te
    return te


def _offsets(sizes):
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


def _statistics(te, pts, sizes, d_y, d_x, k):
    import torch
    got = te.knn_counts(torch.from_numpy(np.ascontiguousarray(pts)).cuda(), _offsets(sizes), d_y, d_x, k)
    return got[0].cpu().numpy(), got[1].cpu().numpy(), got[2]


def _brute_force(p, d_y, k):
    """Radii and counts of one chunk: a coordinate difference that is no number says nothing about
    its pair, and a pair without any in a space lies in no ball of that space."""
    eps = np.empty(p.shape[1], np.float32)
    cnt = np.empty((3, p.shape[1]), np.int32)
    with np.errstate(invalid="ignore"):
        for i in range(p.shape[1]):
            d = np.abs(p - p[:, i:i + 1])
            dt, dp = d[0], np.fmax.reduce(d[1:1 + d_y])
            ds = np.fmax.reduce(d[1 + d_y:])
            dj = np.fmax(np.fmax(dt, dp), ds)
            e = np.sort(np.where(np.isnan(dj), np.float32(np.inf), dj))[k]
            in_p = dp < e
            own = int(e > 0)
            eps[i] = e
            cnt[:, i] = in_p.sum() - own, (in_p & (dt < e)).sum() - own, (in_p & (ds < e)).sum() - own
    return eps, cnt


def _with_nan(kind, N, D, d_y, seed):
    p = normal64(derive_key(seed, N, D), N * D).reshape(D, N)
    if kind == "future":
        p[0, 1::7] = np.nan
    elif kind == "past":
        p[1:1 + d_y, 3::11] = np.nan
    elif kind == "source":
        p[1 + d_y:, 2::9] = np.nan
    elif kind == "points":                   # whole points, as a marker of missing values
        p[:, 5::13] = np.nan
    elif kind == "single":                   # every coordinate somewhere, alone and together, beside infinities
        for m in range(D):
            p[m, m::5 + m] = np.nan
        p[1, 4::17] = np.inf
        p[D - 1, 6::19] = -np.inf
    return p.astype(np.float32)


@pytest.mark.parametrize("d_y,d_x,k", [(1, 1, 4), (3, 3, 4), (2, 1, 7), (4, 2, 12)])
@pytest.mark.parametrize("kind", ["future", "past", "source", "points", "single"])
def test_points_that_are_no_numbers(te, monkeypatch, kind, d_y, d_x, k):
    sizes = [40, 64, 65, 1100]
    pts = _with_nan(kind, sum(sizes), 1 + d_y + d_x, d_y, 601)
    print("nan", kind, d_y, d_x, k, flush=True)
    want = [_brute_force(pts[:, a:b], d_y, k) for a, b in zip(_offsets(sizes)[:-1], _offsets(sizes)[1:])]
    for no_sort in ("0", "1"):
        monkeypatch.setenv("TE_NO_SORT", no_sort)
        eps, cnt, _ = _statistics(te, pts, sizes, d_y, d_x, k)
        np.testing.assert_array_equal(eps, np.concatenate([w[0] for w in want]))
        np.testing.assert_array_equal(cnt, np.concatenate([w[1] for w in want], axis=1))


def _many(kind, d_y, D):
    """30 000 blocks of chunks of one to eighteen blocks: searched by persistent waves, a block each."""
    sizes = [65, 190, 1100, 700, 511] * 714
    pts = _with_nan(kind, sum(sizes[:50]), D, d_y, 602).astype(np.float32)
    if kind == "infinite":
        pts[0, 1::13] = np.inf
        pts[-1, 2::9] = -np.inf
        pts[1, ::7] = np.inf
        pts[1, ::11] = -np.inf
    elif kind == "grid":
        pts = np.round(pts * 2) / 2
    out = np.tile(pts, (1, -(-sum(sizes) // pts.shape[1])))[:, :sum(sizes)]
    return out, sizes


@pytest.mark.parametrize("slots", [4, 8])
@pytest.mark.parametrize("kind,d_y,d_x,k", [("gauss", 2, 2, 4), ("grid", 3, 3, 4), ("grid", 1, 1, 6), ("infinite", 2, 2, 4),
                                            ("infinite", 4, 1, 4), ("points", 2, 2, 4), ("single", 3, 1, 4),
                                            ("single", 1, 2, 9)])
def test_persistent_waves_equal_the_unordered_search(te, monkeypatch, kind, d_y, d_x, k, slots):
    """Single chunks in launches too large for several waves to a block, one and two blocks of
    candidates counted together: radii and counts of the every-pair search."""
    pts, sizes = _many(kind, d_y, 1 + d_y + d_x)
    print("persistent", kind, d_y, d_x, k, slots, flush=True)
    monkeypatch.setenv("TE_SLOTS", str(slots))
    got = _statistics(te, pts, sizes, d_y, d_x, k)
    monkeypatch.setenv("TE_NO_SORT", "1")
    want = _statistics(te, pts, sizes, d_y, d_x, k)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])
    # eq. 9 sums N terms below 14 in another order: N rounding errors of 2^-53 * 14 N at most, over N
    np.testing.assert_allclose(got[2], want[2], rtol=0, atol=14 * max(sizes) * 2.0 ** -53, equal_nan=True)


def _copies(points, S, d_y=2, d_x=2, W=13):
    """`points` copies of one window of 50 W points."""
    wl = synth.generic((6092, S), R=50, T=60, d_y=d_y, d_x=d_x, starts=(30,), windows=(W,), n_surrogates=S)
    wl.window_start = np.full(points, 30, np.int32)
    wl.window_len = np.full(points, W, np.int32)
    wl.trials = np.full(points, 50, np.int32)
    if S:
        wl.perms = np.ascontiguousarray(np.repeat(wl.perms, points, axis=1))
    return wl


def _surrogates(te, wl):
    import torch
    perms = torch.from_numpy(wl.perms).cuda() if wl.n_surrogates else None
    plan = te.Plan.from_workload(wl)
    return plan, plan.surrogates(torch.from_numpy(wl.x).cuda(), torch.from_numpy(wl.y).cuda(), perms)


@pytest.mark.parametrize("d_y,d_x,S,points", [(2, 2, 3, 500), (1, 1, 4, 500), (3, 3, 5, 180), (4, 3, 2, 300), (2, 2, 0, 2300)])
def test_persistent_launches_of_every_shape(te, monkeypatch, d_y, d_x, S, points):
    """Launches of persistent waves, chunk sets and single chunks, in every kind of shape: the
    estimates of the default shape, of single chunks and of one window alone, bit for bit."""
    wl = _copies(points, S, d_y, d_x)
    alone = _surrogates(te, _copies(1, S, d_y, d_x))[1]
    for env in ({}, {"TE_NO_SETS": "1"}, {"TE_SLOTS": "4", "TE_WAVES_PER_WG": "1", "TE_WG_PER_CU": "3"},
                {"TE_SLOTS": "16", "TE_WAVES_PER_WG": "2", "TE_WG_PER_CU": "1"},
                {"TE_SLOTS": "8", "TE_WAVES_PER_WG": "1", "TE_WG_PER_CU": "7"},
                {"TE_SLOTS": "8", "TE_WAVES_PER_WG": "4"}):
        print("shape", d_y, d_x, S, points, env, flush=True)
        with monkeypatch.context() as m:
            for name, v in env.items():
                m.setenv(name, v)
            t0, ts, _ = _surrogates(te, wl)[1]
        np.testing.assert_array_equal(t0, np.full_like(t0, alone[0][0, 0]))
        np.testing.assert_array_equal(ts[0], np.repeat(alone[1][0], points, axis=0))


def test_tuning_times_the_persistent_waves(te):
    """The tuned shape is that of persistent waves; a plan small enough for several waves to a
    block is timed in that form too.  The two forms examine different numbers of pairs: as many
    per window as in a batch of persistent waves."""
    import torch
    n = 2300
    plan, _ = _surrogates(te, _copies(n, 0))
    wl = _copies(1, 0)
    x, y = torch.from_numpy(wl.x).cuda(), torch.from_numpy(wl.y).cuda()
    small = te.Plan.from_workload(wl)
    te.profile_enable(True, work=True)
    try:
        te.profile_work(reset=True)
        plan.surrogates(x, y)
        persistent = te.profile_work(reset=True)
        small.surrogates(x, y)
        shared = te.profile_work(reset=True)
        te.profile_read(reset=True)
        small.autotune(x, y)
        _, launches = te.profile_read(reset=True)
        tuned = te.profile_work(reset=True)
        small.surrogates(x, y)
        after = te.profile_work(reset=True)
    finally:
        te.profile_enable(False)
        te.tune_clear()
    print("pairs", persistent, shared, tuned, launches, after, flush=True)
    assert persistent[0] % n == 0 and persistent[0] // n != shared[0]
    assert tuned[0] == launches * (persistent[0] // n)
    assert after == shared


def _rejections(key, n):
    """Draws of a row of n trials that the first round rejects."""
    s = np.arange(n, 1, -1, dtype=np.uint64)
    low = ((stream_u64(key, n - 1) >> np.uint64(32)) * s) & np.uint64(0xFFFFFFFF)
    return int(np.count_nonzero(low < (np.uint64(1 << 32) - s) % s))


def test_rows_with_rejected_draws_at_the_longest_in_lds(te):
    """Rejected draws redrawn in rows resolved in parallel (up to 8 192 trials) and in order (above)."""
    seed, S, trials = 18, 250, (8191, 8192, 8193)
    held = [sum(_rejections(derive_key(seed, 77, 0, c, s), n) for s in range(S)) for c, n in enumerate(trials)]
    print("rejected draws", held, flush=True)
    assert min(held) >= 1
    wl = synth.configs.Workload(name="perm", x=np.zeros((1, 8193, 12), np.float32), y=np.zeros((1, 8193, 12), np.float32),
                                d_y=1, d_x=1, tau=1, u=1, k=4, window_start=np.ones(3, np.int32),
                                window_len=np.full(3, 8, np.int32), trials=np.array(trials, np.int32), n_surrogates=S)
    wl.perm_seed = seed
    want = synth.configs.make_perms(seed, 1, wl.trials, S, 8193)
    np.testing.assert_array_equal(te.Plan.from_workload(wl).permutations().cpu().numpy(), want)


@pytest.mark.parametrize("d_y,sizes", [(1, [524289, 700]), (3, [9001, 530001, 64])])
def test_spaces_sorted_whole_beside_smaller_ones(te, monkeypatch, d_y, sizes):
    """Above 524 288 points a sort by the first coordinate cuts the slabs, more than 64 of them."""
    pts = normal64(derive_key(603, d_y), sum(sizes) * (2 + d_y)).reshape(2 + d_y, -1).astype(np.float32)
    print("sorted whole", d_y, sizes, flush=True)
    got = _statistics(te, pts, sizes, d_y, 1, 4)
    monkeypatch.setenv("TE_NO_SORT", "1")
    want = _statistics(te, pts, sizes, d_y, 1, 4)
    np.testing.assert_array_equal(got[0], want[0])
    np.testing.assert_array_equal(got[1], want[1])


def test_embedding_choice_over_more_points_than_slabs_hold(te):
    import torch
    from oracle import ragwitz as rg
    R, W = 5243, 100                          # 524 300 points
    y = normal64(derive_key(604), R * (W + 10)).reshape(R, W + 10).astype(np.float32)
    sample = np.unique(np.round(np.linspace(0, R * W - 1, 25)).astype(int))
    print("ragwitz", R * W, flush=True)
    _, pred = te.ragwitz(torch.from_numpy(y).cuda(), 8, W, [(1, 1), (3, 2)], 3, want_pred=True)
    for c, (d, tau) in enumerate([(1, 1), (3, 2)]):
        S, tgt = rg.states(y, d, tau, 8, W)
        np.testing.assert_array_equal(pred[c].cpu().numpy()[sample], rg.predictions_points(S, tgt, 3, sample))


@pytest.mark.parametrize("kind", ["gauss", "grid", "constant"])
@pytest.mark.parametrize("R,W,n", [(1, 18, 3), (3, 43, 1), (16, 16, 2), (3, 910, 3), (3, 911, 3),    # every pair: one and two
                                   (17, 241, 16), (64, 65, 16), (121, 68, 16)])       # references a wave; 8 and 4 waves a block
def test_embedding_choice_at_the_lines_of_its_searches(te, kind, R, W, n):
    import torch
    from oracle import ragwitz as rg
    y = normal64(derive_key(605, R, W), R * (W + 20)).reshape(R, W + 20)
    if kind == "grid":
        y = np.round(y)
    elif kind == "constant":
        y[:] = 2.0
    y = y.astype(np.float32)
    cands = [(8, 1), (3, 2), (1, 1)][:n] if n < 16 else [(d, tau) for d in range(1, 9) for tau in (1, 2)]
    sample = np.unique(np.round(np.linspace(0, R * W - 1, 30)).astype(int))
    for k in (1, 3, 5, 16):
        print("ragwitz", kind, R * W, n, k, flush=True)
        _, pred = te.ragwitz(torch.from_numpy(y).cuda(), 18, W, cands, k, want_pred=True)
        for c in range(0, len(cands), 1 if n < 16 else 5):
            S, tgt = rg.states(y, *cands[c], 18, W)
            np.testing.assert_array_equal(pred[c].cpu().numpy()[sample], rg.predictions_points(S, tgt, k, sample))
