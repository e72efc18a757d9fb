"""GPU tests of te_ragwitz's search over ordered points at the sizes where its blocks, slabs and
launches change: predictions equal the oracle's bit for bit."""
import numpy as np
import pytest

from oracle import ragwitz as rg
from synth.rng import derive_key, normal64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def te():
    import paper_1401_4068_amd as te
    return te


def _series(kind, R, T):
    y = normal64(derive_key(811, R, T), R * T).reshape(R, T)
    for t in range(1, T):
        y[:, t] += 0.5 * y[:, t - 1]
    if kind == "grid":                 # equal distances everywhere: the index ranks them
        y = np.round(y)
    elif kind == "constant":
        y[:] = 2.0
    return y.astype(np.float32)


@pytest.mark.parametrize("kind", ["gauss", "grid", "constant"])
@pytest.mark.parametrize("R,W", [(1, 3), (7, 9), (8, 8), (5, 13), (13, 30), (64, 128), (67, 123), (113, 146)])
def test_predictions_at_the_sizes_of_blocks_and_slabs(te, kind, R, W):
    """2 points per k to one block, blocks with ragged ends, 8 192 and 8 241 points (one slab and
    several), 16 498 points (32-bit maps, codes in the key scratch)."""
    import torch
    y = _series(kind, R, W + 20)
    N = R * W
    cands = [(1, 1), (3, 2), (8, 1)] if N < 1000 else [(1, 1), (2, 3), (5, 1)]
    sample = np.unique(np.round(np.linspace(0, N - 1, 60)).astype(int))
    for k in (1, 2, 8, 16):
        if k >= N:
            continue
        print("ragwitz", kind, N, k, flush=True)
        _, pred = te.ragwitz(torch.from_numpy(y).cuda(), 18, W, cands, k, want_pred=True)
        pred = pred.cpu().numpy()
        for c, (d, tau) in enumerate(cands):
            S, tgt = rg.states(y, d, tau, 18, W)
            np.testing.assert_array_equal(pred[c][sample], rg.predictions_points(S, tgt, k, sample))


def test_more_candidates_than_a_launch_or_the_search_area_takes(te):
    """40 candidates are searched 16 at a time; 24 points leave room for fewer."""
    import torch
    for R, W in ((4, 6), (20, 20)):
        y = _series("gauss", R, W + 60)
        cands = [(d, tau) for tau in range(1, 6) for d in range(1, 9)]
        print("candidates", len(cands), "points", R * W, flush=True)
        scores, pred = te.ragwitz(torch.from_numpy(y).cuda(), 50, W, cands, 3, want_pred=True)
        for c, (d, tau) in enumerate(cands):
            S, tgt = rg.states(y, d, tau, 50, W)
            np.testing.assert_array_equal(pred[c].cpu().numpy(), rg.predictions(S, tgt, 3))
            assert scores[c] == pytest.approx(rg.nmse(tgt, rg.predictions(S, tgt, 3)), rel=1e-12)
