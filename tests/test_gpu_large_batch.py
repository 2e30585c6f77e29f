"""Weight gradients of a large batch, whose sums over the samples average the
sweeps' roundings out and keep what is the same for every sample: the split
weights and the sums' own order.

Bounds, of the norm of a kind's blocks: weights split in two FP16 parts carry a
relative rounding of 3.9e-8 rms, in both directions of four layers; FP64 sweeps
with weights so rounded are off by 0.8e-7 to 1.0e-7 (weights) and 0.9e-7 (output
weights).  FP32 sums of 4096 rows in eight to 64 partials of trees add 3e-8 to
6e-8 in quadrature: 1.25e-7 and 1.1e-7, and a fifth on top.  (Biases: no bound
here; their sums cancel by amounts that depend on the data.)"""
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


@pytest.mark.parametrize("n,width,layers,K,B", [(38, 256, 4, 4, 4096), (38, 256, 4, 1, 4000)])
def test_gradient_of_a_coherent_batch(torch, rid, n, width, layers, K, B):
    widths = [width] * layers
    rng = np.random.default_rng(1)
    s = ridgen.f32(rng.uniform(-np.pi, np.pi, (B, n)))
    a, b = rng.uniform(0.5, 5.0, n), rng.uniform(-np.pi, np.pi, n)
    F = ridgen.f32(a * np.sin(s - b) + rng.normal(0.0, 0.5, s.shape))
    params = ridgen.xavier_ensemble(2 * n, widths, K, 1000, bias_std=0.05)
    E = rid.Ensemble(n, widths, K, params)
    _, grad = rid.mf_loss_grad(E, torch.from_numpy(s).cuda(), torch.from_numpy(F).cuda())
    torch.cuda.synchronize()
    grad = grad.cpu().numpy().reshape(K, -1).astype(np.float64)
    err = {"weights": 0.0, "biases": 0.0, "output": 0.0}
    ref = [O.train_loss_grad(m, s, F)[1] for m in ridgen.unpack_params(params, 2 * n, widths, K)]
    off, prev = 0, 2 * n
    blocks = []
    for w in widths:
        blocks += [("weights", off, w * prev), ("biases", off + w * prev, w)]
        off += w * prev + w
        prev = w
    blocks.append(("output", off, prev))
    flat = np.stack([O.flat_grad(g) for g in ref])
    for name, o, cnt in blocks:
        x, y = grad[:, o:o + cnt], flat[:, o:o + cnt]
        err[name] = max(err[name], np.linalg.norm(x - y) / np.linalg.norm(y))
    print(f"K={K} B={B}: " + ", ".join(f"{k} {v:.2e}" for k, v in err.items()), flush=True)
    assert err["weights"] <= 1.5e-7 and err["output"] <= 1.3e-7


def test_weights_that_round_alike(torch, rid):
    """Every weight's last 13 bits are 0x803: 11 + 11 bits of an FP16 pair leave an
    odd half unit that rounds the same way in every weight (up, 2^-24 to 2^-23 of
    it), so the errors of one rounding add up through the layers: FP64 sweeps with
    weights so rounded are off by 1.4e-7.  With two roundings of opposite error
    over the batch they are off by 0.33e-7.  The bound: that, FP32 sums (up to
    6e-8) and the sweeps' own arithmetic (7e-8) in quadrature, and a fifth on top."""
    n, widths, K, B = 38, [256] * 4, 1, 4096
    rng = np.random.default_rng(1)
    s = ridgen.f32(rng.uniform(-np.pi, np.pi, (B, n)))
    a, b = rng.uniform(0.5, 5.0, n), rng.uniform(-np.pi, np.pi, n)
    F = ridgen.f32(a * np.sin(s - b) + rng.normal(0.0, 0.5, s.shape))
    params = np.array(ridgen.xavier_ensemble(2 * n, widths, K, 1000, bias_std=0.05), np.float32)
    bits = params.view(np.uint32)
    blocks, off, prev = [], 0, 2 * n
    for w in widths:
        blocks.append((off, w * prev))
        bits[off:off + w * prev] = (bits[off:off + w * prev] & ~np.uint32(0x1FFF)) | np.uint32(0x803)
        off += w * prev + w
        prev = w
    E = rid.Ensemble(n, widths, K, params)
    _, grad = rid.mf_loss_grad(E, torch.from_numpy(s).cuda(), torch.from_numpy(F).cuda())
    torch.cuda.synchronize()
    grad = grad.cpu().numpy().reshape(-1).astype(np.float64)
    model, = ridgen.unpack_params(params, 2 * n, widths, K)
    ref = O.flat_grad(O.train_loss_grad(model, s, F)[1])
    x, y = (np.concatenate([g[o:o + c] for o, c in blocks]) for g in (grad, ref))
    err = np.linalg.norm(x - y) / np.linalg.norm(y)
    print(f"weights {err:.2e}", flush=True)
    assert err <= 1.2e-7
