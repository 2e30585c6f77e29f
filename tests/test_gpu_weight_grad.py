"""The weight-gradient products at the edges of their tiles (64 x 64), steps
(16 rows of a half of the stacked slabs), chunks and passes, in both forms
(split FP16 after the fused sweeps, split BF16 after the general ones), against
the FP64 oracle; operand scales of the two halves far apart; and what must not
be finite.

Tolerance: 2e-5 of a member's largest entry.  The operands keep 22 bits, the
accumulators round 24-bit sums of up to 2B / 64 terms per wave, and the sweeps'
own FP32 rounding enters both halves: a few 1e-6 together."""
import numpy as np
import pytest

import ridgen
from oracle import rid_oracle as O

pytestmark = pytest.mark.gpu
TOL = 2e-5


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


def _err(got, ref):
    return max(np.abs(got[k] - ref[k]).max() / np.abs(ref[k]).max() for k in range(len(ref)))


# (n, widths, K, B, general, budget): rows 1, 8, 15 .. 17, 31 .. 33 of a half;
# tiles of 63 .. 65 and 129 columns; batches of one and of several chunks; a
# budget that takes several passes (64 rows each and a last one of 36)
CASES = [
    (2, [65, 1, 129], 2, 1, False, 0), (5, [63, 64], 3, 8, False, 0),
    (5, [64, 65], 1, 15, False, 0), (33, [96, 40], 2, 16, False, 0),
    (32, [129, 33], 2, 17, False, 0), (3, [30, 31, 32, 33], 2, 31, False, 0),
    (16, [128], 1, 32, False, 0), (7, [100] * 3, 4, 33, False, 0),
    (11, [64] * 2, 1, 1025, False, 0), (6, [130, 20], 5, 700, False, 0),
    (4, [48, 52], 2, 100, False, 1), (4, [48, 52], 2, 100, True, 1),
    (2, [65, 1, 129], 2, 1, True, 0), (5, [64, 65], 1, 15, True, 0),
    (33, [96, 40], 2, 16, True, 0), (32, [129, 33], 2, 17, True, 0),
    (7, [100] * 3, 4, 33, True, 0), (11, [64] * 2, 1, 1025, True, 0)]


@pytest.mark.parametrize("n,widths,K,B,general,budget", CASES)
def test_weight_gradient_edges(torch, rid, n, widths, K, B, general, budget):
    params = ridgen.xavier_ensemble(2 * n, widths, K, 40 + n, bias_std=0.1)
    s, F, _ = ridgen.mf_training_set(B, n)
    # (16-bit ensembles train their FP32 masters through the general sweeps)
    E = rid.Ensemble(n, widths, K, params, rid.RID_BF16 if general else rid.RID_FP32)
    if budget:
        E.set_train_budget(budget)
    loss, grad = rid.mf_loss_grad(E, torch.from_numpy(s).cuda(), torch.from_numpy(F).cuda())
    torch.cuda.synchronize()
    ref = [O.train_loss_grad(m, s, F) for m in ridgen.unpack_params(params, 2 * n, widths, K)]
    gerr = _err(grad.cpu().numpy().reshape(K, -1).astype(np.float64),
                np.stack([O.flat_grad(g) for _, g in ref]))
    lerr = np.abs(loss.cpu().numpy() / np.array([l_ for l_, _ in ref]) - 1.0).max()
    print(f"n={n} {widths} K={K} B={B} general={general}: grad {gerr:.2e} loss {lerr:.2e}",
          flush=True)
    assert gerr <= TOL and lerr <= 1e-5


@pytest.mark.parametrize("spread", [1e-12, 1e-6, 1e6])
def test_rows_of_very_different_size(torch, rid, spread):
    """One sample's upstream gradient sets the scale of a whole slab; the
    others' share of the result is lost only where FP32 sums lose it too."""
    n, widths, K, B = 6, [70, 80], 2, 48
    rng = np.random.default_rng(8)
    s = ridgen.f32(rng.uniform(-np.pi, np.pi, (B, n)))
    rho = rng.normal(size=(B, K, n))
    rho[1:] *= spread
    rho = ridgen.f32(rho)
    params = ridgen.xavier_ensemble(2 * n, widths, K, 71, bias_std=0.1)
    E = rid.Ensemble(n, widths, K, params)
    grad = rid.mf_grad(E, torch.from_numpy(s).cuda(), torch.from_numpy(rho).cuda())
    torch.cuda.synchronize()
    ref = np.stack([O.flat_grad(O.mean_force_vjp(m, s, rho[:, k]))
                    for k, m in enumerate(ridgen.unpack_params(params, 2 * n, widths, K))])
    assert _err(grad.cpu().numpy().reshape(K, -1).astype(np.float64), ref) <= TOL


@pytest.mark.parametrize("general", [False, True])
def test_zero_and_not_finite(torch, rid, general):
    n, widths, K, B = 5, [64, 64], 2, 20
    s, F, _ = ridgen.mf_training_set(B, n)
    params = ridgen.xavier_ensemble(2 * n, widths, K, 72, bias_std=0.1)
    E = rid.Ensemble(n, widths, K, params, rid.RID_BF16 if general else rid.RID_FP32)
    rho = torch.zeros(B, K, n).cuda()
    st = torch.from_numpy(s).cuda()
    assert (rid.mf_grad(E, st, rho) == 0).all()
    for bad in (np.inf, np.nan):
        rho[7, 1, 2] = bad
        grad = rid.mf_grad(E, st, rho).reshape(K, -1)
        torch.cuda.synchronize()
        assert (grad[0] == 0).all()
        w1 = grad[1][:widths[0] * 2 * n]
        assert not torch.isfinite(w1).any()
