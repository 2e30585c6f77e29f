"""Saturated units of FP32 ensembles, |z| from 6 to 14 on either side: tanh' is
formed from q = 1 - |tanh| and keeps its precision where 1 - tanh^2 has lost it.

One unit per member, z = b + cos s, so a member's mean force is
-sin s tanh'(z) and its energy tanh(z).  Bounds: tanh'(6) = 2.5e-5, and
2^y of y = z 2/ln 2 (up to 40, rounded to 1.9e-6) is good to a few 1e-6, so
tanh' to 2e-10; the split product's step of 2^-38 lies below that.  tanh to two
units in the last place below 1 (1.2e-7).  The training sweeps form tanh' from
tanh again: twice tanh's half unit (3e-8) and a rounding, 1.2e-7."""
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


def _members(K):
    """One unit each: W = (1, 0), |b| from 7 to 13, w_o = 1."""
    b = np.linspace(7.0, 13.0, K // 2)
    b = np.concatenate([-b, b])
    params = ridgen.f32(ridgen.pack_params(
        [([np.array([[1.0, 0.0]])], [np.array([x])], np.array([1.0]), 0.0) for x in b]))
    return params, ridgen.unpack_params(params, 2, [1], K)


def test_mean_force_through_saturated_units(torch, rid):
    K, B = 64, 200
    params, models = _members(K)
    s = ridgen.f32(np.random.default_rng(0).uniform(0.2, np.pi - 0.2, (B, 1)))
    out = rid.model_dev(rid.Ensemble(1, [1], K, params), torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    A, _ = O.ensemble_mean_force(models, s.astype(np.float64))
    z = np.array([m[1][0][0] for m in models])[None, :] + np.cos(s.astype(np.float64))
    g = -np.sin(s.astype(np.float64)) / np.cosh(z) ** 2
    gg, Ag = out[3].cpu().numpy()[:, :, 0], out[2].cpu().numpy()
    err, errA = np.abs(gg - g).max(), np.abs(Ag - A).max()
    print(f"tanh' {err:.2e}, tanh {errA:.2e}", flush=True)
    assert err <= 2e-10 and errA <= 1.2e-7


def test_training_gradient_through_saturated_units(torch, rid):
    """dJ/dw_o of a single sample is -sin s tanh'(z)."""
    K = 64
    params, models = _members(K)
    E = rid.Ensemble(1, [1], K, params)
    worst = 0.0
    for s0 in np.linspace(0.2, np.pi - 0.2, 25):
        s = ridgen.f32(np.full((1, 1), s0))
        grad = rid.mf_grad(E, torch.from_numpy(s).cuda(),
                           torch.ones((1, K, 1), dtype=torch.float32, device="cuda"))
        torch.cuda.synchronize()
        got = grad.cpu().numpy().reshape(K, -1)[:, 3]      # W (2), b, w_o, b_o
        x = float(s[0, 0])
        z = np.array([m[1][0][0] for m in models]) + np.cos(x)
        worst = max(worst, np.abs(got + np.sin(x) / np.cosh(z) ** 2).max())
    print(f"tanh' in the training sweeps: {worst:.2e}", flush=True)
    assert worst <= 1.2e-7


def test_members_and_walkers_that_are_not_finite(torch, rid):
    """Infinite biases saturate exactly; a NaN stays a NaN."""
    b = [np.inf, -np.inf, np.nan, 200.0, -200.0]
    params = ridgen.f32(ridgen.pack_params(
        [([np.array([[1.0, 0.0]])], [np.array([x])], np.array([1.0]), 0.0) for x in b]))
    s = torch.tensor([[0.3], [2.0]], dtype=torch.float32).cuda()
    _, _, A, g = rid.model_dev(rid.Ensemble(1, [1], len(b), params), s)
    A, g = A.cpu().numpy(), g.cpu().numpy()[:, :, 0]
    keep = [0, 1, 3, 4]
    assert np.array_equal(A[:, keep], np.tile(np.float32([1, -1, 1, -1]), (2, 1)))
    assert not g[:, keep].any()
    assert np.isnan(A[:, 2]).all() and np.isnan(g[:, 2]).all()
