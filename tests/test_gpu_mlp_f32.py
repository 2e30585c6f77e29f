"""GPU parity of the FP32 MLP kernel's instantiations (padded widths 64, 128,
192, 256, 320, 384, 512; 16, 32 and 64 walkers per workgroup) against the FP64
oracle at the edges of its tiles, the same bits whatever tile a walker lands
in, and the operand scales of the split products: output weights far from 1,
raw CVs far from 1, walkers with NaN CVs.

Tolerance: the FP32 path's 1e-5 (normwise per walker), as everywhere."""
import numpy as np
import pytest

import ridgen
from oracle import rid_oracle as O
from tests.gpu_common import FP32_TOL

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


def _run(torch, rid, n, widths, K, params, s, mask=None, resnet=False):
    E = rid.Ensemble(n, widths, K, params)
    if mask is not None:
        E.set_angular_mask(mask)
    if resnet:
        E.set_resnet(True)
    out = rid.model_dev(E, torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


def _check(n, widths, K, params, s, got, mask=None, resnet=False):
    models = ridgen.unpack_params(params, 2 * n, widths, K)
    if resnet:
        models = [m + (True,) for m in models]
    A, g = O.ensemble_mean_force(models, s.astype(np.float64), mask)
    _, _, Ag, gg = got
    err = np.abs(gg - g).max(axis=2) / np.abs(g).max(axis=2)
    errA = np.abs(Ag - A).max() / np.abs(A).max()
    print(f"n={n} {widths} K={K} B={len(s)}: g {err.max():.2e}, A {errA:.2e}", flush=True)
    assert err.max() <= FP32_TOL and errA <= FP32_TOL


# (n_cv, widths, K, B, residual): each padded width below, at and above its
# edge; 1, 15, 17, 33 and 65 walkers end in ragged tiles of 16, 32 and 64
# rows; the large B take 32 rows (250+ workgroups of 16) and 64
@pytest.mark.parametrize("n,widths,K,B,resnet", [
    (1, [1], 1, 1, False), (3, [63, 64], 2, 15, False), (16, [65, 3, 40], 3, 17, False),
    (17, [128] * 6, 2, 33, False), (38, [129] * 4, 4, 65, False), (33, [192] * 3, 5, 1030, False),
    (38, [193] * 4, 3, 1400, False), (48, [256] * 2, 4, 2065, False),
    (20, [257] * 4, 4, 1300, False), (18, [320] * 4, 4, 12, True), (18, [300] * 3, 4, 1300, True),
    (9, [321] * 4, 2, 31, False), (40, [384] * 3, 4, 1300, True), (60, [385] * 2, 2, 47, False),
    (64, [512] * 5, 2, 17, False), (120, [512] * 3, 4, 1030, False), (200, [130] * 2, 2, 40, False),
    (256, [512] * 2, 2, 35, False), (30, [512] * 4, 2, 20, True)])
def test_model_dev_parity_at_tile_edges(torch, rid, n, widths, K, B, resnet):
    rng = np.random.default_rng(n + B)
    s = ridgen.f32(rng.uniform(-np.pi, np.pi, (B, n)))
    params = ridgen.xavier_ensemble(2 * n, widths, K, 300 + n, bias_std=0.1)
    got = _run(torch, rid, n, widths, K, params, s, resnet=resnet)
    sel = np.unique(np.concatenate([np.arange(min(B, 20)), np.arange(max(0, B - 40), B)]))
    _check(n, widths, K, params, s[sel], [o[sel] for o in got], resnet=resnet)


@pytest.mark.parametrize("n,widths,K,B,resnet", [
    (38, [64] * 3, 4, 9000, False), (38, [100] * 3, 4, 2000, False), (38, [256] * 4, 4, 2000, False),
    (38, [256] * 4, 4, 4500, False), (18, [300] * 4, 4, 1300, True), (38, [512] * 3, 4, 1100, False)])
def test_same_bits_in_every_row_tile(torch, rid, n, widths, K, B, resnet):
    """A large call (32 or 64 rows a workgroup) and calls on its slices (16
    rows, other places in the tile) give the same bits."""
    rng = np.random.default_rng(5)
    s = ridgen.f32(rng.uniform(-np.pi, np.pi, (B, n)))
    params = ridgen.xavier_ensemble(2 * n, widths, K, 77, bias_std=0.1)
    full = _run(torch, rid, n, widths, K, params, s, resnet=resnet)
    for lo, hi in ((0, 1), (37, 96), (B - 33, B)):
        part = _run(torch, rid, n, widths, K, params, np.ascontiguousarray(s[lo:hi]), resnet=resnet)
        for a, b in zip(full, part):
            assert np.array_equal(a[lo:hi], b)


@pytest.mark.parametrize("factor", [2.0 ** 60, 2.0 ** -60, 3.7e4])
@pytest.mark.parametrize("resnet", [False, True])
def test_output_weights_far_from_one(torch, rid, factor, resnet):
    """The mean force is linear in the output weights, whatever their size."""
    n, widths, K, B = 12, [96] * 4, 3, 50
    s = ridgen.f32(np.random.default_rng(1).uniform(-np.pi, np.pi, (B, n)))
    models = ridgen.unpack_params(ridgen.xavier_ensemble(2 * n, widths, K, 9, bias_std=0.1),
                                  2 * n, widths, K)
    params = ridgen.f32(ridgen.pack_params([(W, b, wo * factor, 0.0) for W, b, wo, _ in models]))
    got = _run(torch, rid, n, widths, K, params, s, resnet=resnet)
    _check(n, widths, K, params, s, got, resnet=resnet)


def test_zero_output_weights_give_zero_forces(torch, rid):
    n, widths, K, B = 6, [70] * 3, 2, 20
    s = ridgen.f32(np.random.default_rng(2).uniform(-np.pi, np.pi, (B, n)))
    models = ridgen.unpack_params(ridgen.xavier_ensemble(2 * n, widths, K, 4), 2 * n, widths, K)
    params = ridgen.f32(ridgen.pack_params([(W, b, wo * 0, 0.25) for W, b, wo, _ in models]))
    eps, gbar, A, g = _run(torch, rid, n, widths, K, params, s)
    assert not g.any() and not eps.any() and np.all(A == np.float32(0.25))


@pytest.mark.parametrize("size", [1e-3, 50.0, 2e4])
def test_raw_cvs_far_from_one(torch, rid, size):
    """Raw CVs of any size share a row with cosines and sines (their weights
    scaled so that the units stay out of saturation)."""
    n, widths, K, B = 80, [100, 100], 2, 40
    rng = np.random.default_rng(8)
    mask = (np.arange(n) % 5 != 0).astype(np.uint8)
    s = rng.uniform(-np.pi, np.pi, (B, n))
    s[:, mask == 0] = rng.uniform(0.3, 1.5, (B, int((mask == 0).sum()))) * size
    s = ridgen.f32(s)
    models = []
    for Ws, bs, wo, bo in ridgen.unpack_params(
            ridgen.xavier_ensemble(2 * n, widths, K, 21, bias_std=0.1), 2 * n, widths, K):
        Ws = [w.copy() for w in Ws]
        Ws[0][:, :n][:, mask == 0] /= max(size, 1.0)
        models.append((Ws, bs, wo, bo))
    params = ridgen.f32(ridgen.pack_params(models))
    _check(n, widths, K, params, s, _run(torch, rid, n, widths, K, params, s, mask=mask), mask=mask)


def test_nan_walker_stays_alone(torch, rid):
    n, widths, K, B = 38, [256] * 4, 4, 64
    s = ridgen.f32(np.random.default_rng(6).uniform(-np.pi, np.pi, (B, n)))
    params = ridgen.xavier_ensemble(2 * n, widths, K, 33, bias_std=0.1)
    ref = _run(torch, rid, n, widths, K, params, s)
    bad = s.copy()
    bad[21, 3] = np.nan
    got = _run(torch, rid, n, widths, K, params, bad)
    keep = np.arange(B) != 21
    for a, b in zip(ref, got):
        assert np.array_equal(a[keep], b[keep])
    assert np.isnan(got[0][21]) and np.isnan(got[2][21]).all() and np.isnan(got[3][21]).all()
