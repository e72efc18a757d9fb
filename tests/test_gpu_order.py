"""GPU tests of the ordered search spaces: at the sizes where the ordering, its slabs and its
blocks of 64 points can go wrong, radii and counts equal those of the unordered search
(TE_NO_SORT=1, which examines every pair) bit for bit."""
import numpy as np
import pytest

import synth
from synth.rng import derive_key, normal64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def te():
    import paper_1401_4068_amd as te
    return te


def _points(kind, N, D, seed):
    p = normal64(derive_key(seed, N, D), N * D).reshape(D, N)
    if kind == "grid":                       # few distinct values: ties in every coordinate and distance
        p = np.round(p * 2) / 2
    elif kind == "constant":                 # the target past says nothing about who is near
        p[1:] = 1.5
        p[-1] = normal64(derive_key(seed, N, 77), N)
    elif kind == "offset":                   # values that share sign, exponent and most of the mantissa
        p = 1.0e6 + p
    elif kind == "tails":                    # a few values far from all others
        p = np.sign(p) * np.abs(p) ** 9
    elif kind == "infinite":                 # unbounded values in every block of coordinates
        p[0, 1::13] = np.inf
        p[-1, 2::9] = -np.inf
        p[1, ::7] = np.inf
        p[1, ::11] = -np.inf
        p[2, 3::5] = np.inf
    return p.astype(np.float32)


def _both(te, monkeypatch, pts, sizes, d_y, d_x, k):
    import torch
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    dev = torch.from_numpy(np.ascontiguousarray(pts)).cuda()
    got = te.knn_counts(dev, off, d_y, d_x, k)
    monkeypatch.setenv("TE_NO_SORT", "1")
    ref = te.knn_counts(dev, off, d_y, d_x, k)
    monkeypatch.delenv("TE_NO_SORT")
    np.testing.assert_array_equal(got[0].cpu().numpy(), ref[0].cpu().numpy())
    np.testing.assert_array_equal(got[1].cpu().numpy(), ref[1].cpu().numpy())
    # eq. 9 sums N terms below 14 in another order: N rounding errors of 2^-53 * 14 N at most, over N
    np.testing.assert_allclose(got[2], ref[2], rtol=0, atol=14 * max(sizes) * 2.0 ** -53, equal_nan=True)


@pytest.mark.parametrize("d_y,d_x,k", [(1, 1, 4), (2, 3, 4), (3, 3, 4), (4, 4, 4), (4, 2, 7)])
@pytest.mark.parametrize("kind", ["gauss", "grid", "constant", "offset", "tails", "infinite"])
def test_ordered_equals_unordered(te, monkeypatch, kind, d_y, d_x, k):
    """One block and its neighbours, a ragged last block, the largest space of one workgroup and
    the smallest of two slabs, the 16-bit map's largest space and the smallest above it."""
    sizes = [9, 63, 64, 65, 128, 129, 1000, 4097, 8191, 8192, 8193, 12001]
    if d_y in (1, 3):
        sizes += [16383, 16384, 16385]
    print(kind, d_y, d_x, k, flush=True)
    _both(te, monkeypatch, _points(kind, sum(sizes), 1 + d_y + d_x, 501), sizes, d_y, d_x, k)


@pytest.mark.parametrize("N,d_y", [(40001, 1), (70003, 2), (33000, 4)])
def test_ordered_equals_unordered_many_slabs(te, monkeypatch, N, d_y):
    print("many slabs", N, d_y, flush=True)
    _both(te, monkeypatch, _points("gauss", N, 2 + d_y, 502), [N], d_y, 1, 4)


@pytest.mark.parametrize("N", [524289, 530001])
def test_ordered_equals_unordered_beyond_slabs(te, monkeypatch, N):
    """More points than slabs of one workgroup each hold: the network sort in global scratch."""
    print("beyond slabs", N, flush=True)
    _both(te, monkeypatch, _points("gauss", N, 4, 503), [N], 2, 1, 4)


def _repeated(points, S, k):
    """`points` copies of one window (650 points: 11 blocks, the last ragged)."""
    wl = synth.generic((6091, S, k), R=50, T=60, d_y=2, d_x=2, k=k, starts=(30,), windows=(13,), n_surrogates=S)
    wl.window_start = np.full(points, 30, np.int32)
    wl.window_len = np.full(points, 13, np.int32)
    wl.trials = np.full(points, 50, np.int32)
    if S:
        wl.perms = np.ascontiguousarray(np.repeat(wl.perms, points, axis=1))
    return wl


@pytest.mark.parametrize("S,k,points", [(0, 4, (1, 50, 300, 2300)), (3, 4, (1, 100, 200)), (0, 3, (1, 100, 300, 2300)),
                                        (0, 6, (1, 200, 500, 800)), (0, 8, (1, 100)), (0, 15, (1, 50)), (0, 4, (1, 600)),
                                        (0, 8, (1, 1500, 1800)), (3, 4, (1, 500))])
def test_estimates_do_not_depend_on_the_waves_per_block(te, S, k, points):
    """The same window alone and among copies of itself, in launches of few and of many blocks
    (8, 4, 2 waves to a block, persistent waves): every estimate has the same bits."""
    import torch
    first = None
    for n in points:
        wl = _repeated(n, S, k)
        print("copies", n, "S", S, "k", k, flush=True)
        x, y = torch.from_numpy(wl.x).cuda(), torch.from_numpy(wl.y).cuda()
        perms = torch.from_numpy(wl.perms).cuda() if S else None
        t0, ts, _ = te.Plan.from_workload(wl).surrogates(x, y, perms)
        first = first or (t0[0, 0], ts[0, 0].copy())
        np.testing.assert_array_equal(t0, np.full_like(t0, first[0]))
        np.testing.assert_array_equal(ts[0], np.repeat(first[1][None], n, axis=0))


@pytest.mark.parametrize("R,trials,S,seed", [(1, (1,), 3, 5), (2, (2, 1), 5, 6), (3, (3, 2), 5, 7),
                                             (257, (63, 64, 65, 256, 257), 9, 8), (2000, (1999, 2000), 6, 9),
                                             (6145, (6143, 6144, 6145), 4, 10), (6144, (6144,), 600, 11)])
def test_drawn_permutations_at_the_edges(te, R, trials, S, seed):
    """Rows of one trial up to the longest drawn across lanes and the next one; 600 rows of 6 144
    trials hold rejected draws (a row has one with probability 0.0022)."""
    C = len(trials)
    print("permutations", R, trials, S, flush=True)
    wl = synth.configs.Workload(name="perm", x=np.zeros((1, R, 12), np.float32), y=np.zeros((1, R, 12), np.float32),
                                d_y=1, d_x=1, tau=1, u=1, k=4, window_start=np.ones(C, np.int32),
                                window_len=np.full(C, 8, np.int32), trials=np.array(trials, np.int32), n_surrogates=S)
    wl.perm_seed = seed
    want = synth.configs.make_perms(seed, 1, wl.trials, S, R)
    np.testing.assert_array_equal(te.Plan.from_workload(wl).permutations().cpu().numpy(), want)
