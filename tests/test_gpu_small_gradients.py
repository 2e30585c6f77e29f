"""Weight gradients of units and inputs far smaller than their layer's largest
keep their own relative precision (Adam normalises every entry by itself):
units whose path to the output is scaled by 2^-k get gradient rows exactly
2^-k as large, bit for bit as precise as their neighbours'; and a unit that an
outlier sample does not move.

Tolerance: the sweeps' gradient bound, 1e-4 of a row's own largest entry."""
import numpy as np
import pytest

import ridgen
from oracle import rid_oracle as O

pytestmark = pytest.mark.gpu
ROW_TOL = 1e-4


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


def _layers(flat, n, widths):
    """The layers' weight gradients [out][in] of one member's packed block."""
    out, off, prev = [], 0, 2 * n
    for w in widths:
        out.append(flat[off:off + w * prev].reshape(w, prev))
        off += w * prev + w
        prev = w
    return out


def _row_err(got, ref):
    return (np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)).max()


@pytest.mark.parametrize("k", [12, 26, 40])
@pytest.mark.parametrize("n,widths,B", [(5, [64, 70], 40), (9, [100] * 3, 700), (18, [300] * 2, 33)])
def test_rows_of_units_with_small_outputs(torch, rid, n, widths, B, k):
    K, f = 2, 2.0 ** -k
    small = slice(3, None, 7)                     # every seventh unit of each layer
    models = []
    for Ws, bs, wo, bo in ridgen.unpack_params(
            ridgen.xavier_ensemble(2 * n, widths, K, 61, bias_std=0.1), 2 * n, widths, K):
        Ws, wo = [w.copy() for w in Ws], wo.copy()
        for W in Ws[1:]:
            W[:, small] *= f
        wo[small] *= f
        models.append((Ws, bs, wo, bo))
    params = ridgen.f32(ridgen.pack_params(models))
    rng = np.random.default_rng(5)
    s = ridgen.f32(rng.uniform(-np.pi, np.pi, (B, n)))
    rho = ridgen.f32(rng.normal(size=(B, K, n)))
    E = rid.Ensemble(n, widths, K, params)
    grad = rid.mf_grad(E, torch.from_numpy(s).cuda(), torch.from_numpy(rho).cuda())
    torch.cuda.synchronize()
    grad = grad.cpu().numpy().reshape(K, -1).astype(np.float64)
    worst = 0.0
    for m, model in enumerate(ridgen.unpack_params(params, 2 * n, widths, K)):
        ref = O.flat_grad(O.mean_force_vjp(model, s, rho[:, m]))
        for got, want in zip(_layers(grad[m], n, widths), _layers(ref, n, widths)):
            worst = max(worst, _row_err(got, want))
    print(f"2^-{k} n={n} {widths} B={B}: rows {worst:.2e}", flush=True)
    assert worst <= ROW_TOL


@pytest.mark.parametrize("size", [2.0 ** 20, 2.0 ** 36])
def test_units_an_outlier_does_not_move(torch, rid, size):
    """Sample 0's upstream gradient is `size` times the others', and it
    saturates the first eight units of the first layer to where tanh' is 0:
    their rows hold the other samples only."""
    n, widths, K, B = 4, [64, 64], 1, 33
    Ws, bs, wo, bo = ridgen.unpack_params(
        ridgen.xavier_ensemble(2 * n, widths, K, 66, bias_std=0.1), 2 * n, widths, K)[0]
    Ws = [w.copy() for w in Ws]
    rng = np.random.default_rng(7)
    s = rng.uniform(-1.0, 1.0, (B, n))
    s[0] = [np.pi, 0.1, 0.2, 0.3]                 # cos s_0 = -1
    Ws[0][:8, :] *= 0.1
    Ws[0][:8, 0] += 20.0                          # z = 20 cos s_0 - 17: -37 at sample 0
    bs = [b.copy() for b in bs]
    c = np.cos(s[1:, 0])
    # (the others stay in reach: cos s_0 within 0.05 of 0.85)
    s[1:, 0] = np.arccos(0.85 + 0.05 * (c - c.mean()) / np.abs(c - c.mean()).max())
    bs[0][:8] = -17.0
    s = ridgen.f32(s)
    params = ridgen.f32(ridgen.pack_params([(Ws, bs, wo, bo)]))
    model = ridgen.unpack_params(params, 2 * n, widths, K)[0]
    rho = rng.normal(size=(B, K, n))
    rho[0] *= size
    rho = ridgen.f32(rho)
    E = rid.Ensemble(n, widths, K, params)
    grad = rid.mf_grad(E, torch.from_numpy(s).cuda(), torch.from_numpy(rho).cuda())
    torch.cuda.synchronize()
    ref = _layers(O.flat_grad(O.mean_force_vjp(model, s, rho[:, 0])), n, widths)[0]
    got = _layers(grad.cpu().numpy().astype(np.float64), n, widths)[0]
    err = _row_err(got[:8], ref[:8])
    print(f"outlier 2^{int(np.log2(size))}: rows of the unmoved units {err:.2e}", flush=True)
    assert err <= ROW_TOL
