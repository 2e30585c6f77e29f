"""The clustering's rounds at their edges, bit-exact against the oracle: mask
words (64 frames), windows (the first 1024, 960, 512, 192 or 128 unmatched
frames for 1, 38, 70, 190 and 256 CVs), batches of 1024 mask words, more
leaders per round than the match kernel stages at a time (16), caps that fill
inside a window, on its last frame and between rounds, and frames with NaNs.

Whole numbers: no tolerance."""
import numpy as np
import pytest

import ridgen
from oracle import rid_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def rid():
    import paper_2408_14070_amd as r
    r.lib()
    return r


def _check(torch, rid, s, t, keep=None, cap=None):
    eps = None
    if keep is not None:
        eps = torch.from_numpy(np.where(keep, 1.0, 0.0).astype(np.float32)).cuda()
    labels, leaders, n = O.leader_cluster(s, t, keep, cap)
    out = rid.cluster_frames(torch.from_numpy(s).cuda(), t, eps=eps, eps0=0.5,
                             max_clusters=cap or len(s))
    torch.cuda.synchronize()
    assert out["n_clusters"] == n
    assert out["leaders"].cpu().numpy().tolist()[:len(leaders)] == leaders
    assert np.array_equal(out["labels"].cpu().numpy(), labels)
    return n


# (B, n, threshold, kept share): few and many clusters, windows filled exactly
# and by one more, whole mask words left out
@pytest.mark.parametrize("B,n,t,share", [
    (1, 1, 0.1, 1.0), (63, 1, 0.05, 1.0), (64, 2, 0.3, 1.0), (65, 2, 0.3, 0.5), (1024, 1, 0.02, 1.0),
    (1025, 1, 0.02, 1.0), (960, 38, 1.0, 1.0), (961, 38, 1.0, 1.0), (2500, 38, 0.9, 0.6),
    (1500, 70, 1.5, 1.0), (700, 190, 2.5, 1.0), (129, 256, 2.0, 1.0), (400, 256, 3.0, 0.9),
    (1000, 7, 0.05, 1.0)])
def test_rounds_match_the_oracle(torch, rid, B, n, t, share):
    s = ridgen.exploration_frames(10, (B + 9) // 10, n, 25, 0.3, seed=B + n)[:B].copy()
    keep = None
    if share < 1.0:
        keep = np.random.default_rng(B).uniform(size=B) < share
        keep[64:192] = False               # whole mask words
    print(f"B={B} n={n} t={t}: {_check(torch, rid, s, t, keep)} clusters", flush=True)


@pytest.mark.parametrize("cap", [1, 2, 15, 16, 17, 40])
def test_caps(torch, rid, cap):
    s = ridgen.exploration_frames(20, 150, 38, 60, 0.3, seed=4)
    _check(torch, rid, s, 3.0, None, cap)


def test_many_words_and_late_frames(torch, rid):
    """More than one batch of 1024 mask words, the kept frames far apart."""
    rng = np.random.default_rng(9)
    s = rng.uniform(-np.pi, np.pi, (140000, 3)).astype(np.float32)
    keep = np.zeros(len(s), bool)
    keep[rng.choice(len(s), 1500, replace=False)] = True
    keep[[0, 65535, 65536, 131071, 131072, 139999]] = True
    _check(torch, rid, s, 0.7, keep)


def test_nan_frames_found_their_own_clusters(torch, rid):
    s = ridgen.exploration_frames(4, 100, 12, 6, 0.3, seed=2)
    s[[5, 70, 333]] = np.nan
    n = _check(torch, rid, s, 1.5)
    assert n >= 3


@pytest.mark.parametrize("lower,upper", [(30, 45), (3, 5), (1, 1), (300, 400), (60, 60)])
def test_adapted_thresholds(torch, rid, lower, upper):
    """Slots past the window are abandoned; the outcome is the rule's."""
    s = ridgen.exploration_frames(10, 80, 38, 40, 0.3, seed=7)
    cap = upper + 6
    t, (labels, leaders, n) = O.adapt_threshold(s, 2.6, lower, upper, None, cap)
    out = rid.cluster_frames(torch.from_numpy(s).cuda(), 2.6, adapt=True, lower=lower, upper=upper,
                             max_clusters=cap)
    torch.cuda.synchronize()
    assert out["threshold"] == t and out["n_clusters"] == n
    assert out["leaders"].cpu().numpy().tolist()[:len(leaders)] == leaders
    assert np.array_equal(out["labels"].cpu().numpy(), labels)


def test_rule_ending_past_the_window(torch, rid):
    """Duplicate-free frames and a window of one cluster between two counts the
    thresholds jump over: the rule runs out of adjustments, and the count and
    labels are those of its last threshold clustered to the end."""
    s = np.repeat(np.array([[0.0], [0.5], [1.0], [1.5]], np.float32), 30, axis=0)
    t, (labels, leaders, n) = O.adapt_threshold(s, 0.4, 3, 3, None, 10)
    out = rid.cluster_frames(torch.from_numpy(s).cuda(), 0.4, adapt=True, lower=3, upper=3,
                             max_clusters=10)
    torch.cuda.synchronize()
    assert n != 3
    assert out["threshold"] == t and out["n_clusters"] == n
    assert np.array_equal(out["labels"].cpu().numpy(), labels)
