"""Raw CVs (distances and the like) of any size beside angular ones in FP32
ensembles: 1e-6 to 1e7, the weights of their columns scaled so that the units
stay out of saturation, evaluation, training gradients and conservative
switching's Hessian-vector products.  The angular part keeps the precision it
has without them, so each group of results is compared by itself.

Tolerances: those of the same calls elsewhere (forces 1e-5, training gradients
1e-4, normwise), here for the angular and the raw columns separately."""
import numpy as np
import pytest

import ridgen
from oracle import rid_oracle as O
from tests.gpu_common import FP32_TOL
from tests.test_gpu_conservative import assert_walkers, walker_bounds

pytestmark = pytest.mark.gpu
GRAD_TOL = 1e-4


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


def _case(n, widths, K, B, size, seed, resnet, every=5):
    """s, mask, params, oracle models: every fifth CV raw, about `size` large."""
    rng = np.random.default_rng(seed)
    mask = (np.arange(n) % every != 0).astype(np.uint8)
    s = rng.uniform(-np.pi, np.pi, (B, n))
    s[:, mask == 0] = rng.uniform(0.3, 1.5, (B, int((mask == 0).sum()))) * size
    s = ridgen.f32(s)
    models = []
    for Ws, bs, wo, bo in ridgen.unpack_params(
            ridgen.xavier_ensemble(2 * n, widths, K, 21, bias_std=0.1), 2 * n, widths, K):
        Ws = [w.copy() for w in Ws]
        Ws[0][:, :n][:, mask == 0] /= size
        models.append((Ws, bs, wo, bo))
    params = ridgen.f32(ridgen.pack_params(models))
    models = ridgen.unpack_params(params, 2 * n, widths, K)
    return s, mask, params, [m + (True,) for m in models] if resnet else models


def _ensemble(rid, n, widths, K, params, mask, resnet):
    E = rid.Ensemble(n, widths, K, params)
    E.set_angular_mask(mask)
    if resnet:
        E.set_resnet(True)
    return E


def _rel(got, ref, axis):
    return (np.abs(got - ref).max(axis=axis) / np.abs(ref).max(axis=axis)).max()


SIZES = [1e-6, 1e-3, 1.0, 1e5, 1e6, 1e7]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("n,widths,K,B,resnet", [
    (80, [100, 100], 2, 40, False), (6, [64], 3, 17, False), (18, [300] * 3, 4, 20, True),
    (40, [256] * 4, 4, 1100, False), (10, [512] * 2, 2, 40, False)])
def test_mean_forces(torch, rid, n, widths, K, B, resnet, size):
    s, mask, params, models = _case(n, widths, K, B, size, 8, resnet)
    out = rid.model_dev(_ensemble(rid, n, widths, K, params, mask, resnet),
                        torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    sel = np.arange(max(0, B - 40), B)
    A, g = O.ensemble_mean_force(models, s[sel].astype(np.float64), mask)
    Ag, gg = out[2].cpu().numpy()[sel], out[3].cpu().numpy()[sel]
    ang, raw = mask == 1, mask == 0
    e_a, e_r = _rel(gg[..., ang], g[..., ang], 2), _rel(gg[..., raw], g[..., raw], 2)
    e_A = np.abs(Ag - A).max() / np.abs(A).max()
    print(f"size {size:g} n={n} {widths}: angular {e_a:.2e} raw {e_r:.2e} A {e_A:.2e}", flush=True)
    assert max(e_a, e_r, e_A) <= FP32_TOL


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("n,widths,K,B,resnet", [
    (20, [100, 90], 2, 40, False), (7, [64], 2, 19, False), (18, [300] * 3, 2, 20, True),
    (40, [200, 256], 4, 1030, False), (100, [64] * 2, 2, 35, False)])
def test_training_gradients(torch, rid, n, widths, K, B, resnet, size):
    """Upstream gradients of the size a fit of labels gives: a raw CV's mean
    force is 1 / size, and so is its residual."""
    s, mask, params, models = _case(n, widths, K, B, size, 9, resnet)
    rng = np.random.default_rng(3)
    rho = rng.normal(size=(B, K, n))
    rho[..., mask == 0] /= size
    rho = ridgen.f32(rho)
    E = _ensemble(rid, n, widths, K, params, mask, resnet)
    grad = rid.mf_grad(E, torch.from_numpy(s).cuda(), torch.from_numpy(rho).cuda())
    torch.cuda.synchronize()
    grad = grad.cpu().numpy().reshape(K, -1).astype(np.float64)
    ref = np.stack([O.flat_grad(O.mean_force_vjp(m, s, rho[:, k], mask=mask))
                    for k, m in enumerate(models)])
    w1, cols = widths[0] * 2 * n, np.concatenate([mask == 1, mask == 1])
    a, b = (x[:, :w1].reshape(K, widths[0], 2 * n) for x in (grad, ref))
    e_a = _rel(a[..., cols], b[..., cols], (1, 2))
    raw = np.concatenate([mask == 0, np.zeros(n, bool)])
    e_r = _rel(a[..., raw], b[..., raw], (1, 2))
    none = np.concatenate([np.zeros(n, bool), mask == 0])   # the raw CVs' second slots
    e_o = _rel(grad[:, w1:], ref[:, w1:], 1)
    print(f"size {size:g} n={n} {widths}: angular {e_a:.2e} raw {e_r:.2e} rest {e_o:.2e}", flush=True)
    assert not a[..., none].any()
    assert max(e_a, e_r, e_o) <= GRAD_TOL


@pytest.mark.parametrize("length", [1.0, 1e2, 1e4, 1e5])
@pytest.mark.parametrize("widths,resnet", [([96] * 3, False), ([300] * 2, True), ([64], False)])
def test_conservative_forces(torch, rid, widths, resnet, length):
    """A chain in other units of length: distances scale, torsions do not, and
    neither does the bias energy, so forces scale with 1 / length."""
    sys_ = ridgen.with_distances(ridgen.chain_system(10, 10), 5)
    n, K, B = sys_.n_cv, 4, 30
    pos1 = ridgen.f32(ridgen.chain_coords(sys_, B, 31))
    pos = ridgen.f32(pos1.astype(np.float64) * length)
    mask = sys_.mask
    base = ridgen.unpack_params(ridgen.xavier_ensemble(2 * n, widths, K, 41, bias_std=0.1),
                                2 * n, widths, K)
    models = []
    for Ws, bs, wo, bo in base:
        Ws = [w.copy() for w in Ws]
        Ws[0][:, :n][:, mask == 0] /= length
        models.append((Ws, bs, wo, bo))
    params = ridgen.f32(ridgen.pack_params(models))
    models = ridgen.unpack_params(params, 2 * n, widths, K)
    if resnet:
        models = [m + (True,) for m in models]
    E = _ensemble(rid, n, widths, K, params, mask, resnet)
    S = rid.System(sys_.n_atoms, sys_.quads, mask)
    eps = O.bias_force(pos.astype(np.float64), sys_.quads, models, 1e30, 2e30, mask=mask)["eps"]
    e0, e1 = 0.5 * eps.min(), 2.0 * eps.max()
    ref = O.bias_force_conservative(pos.astype(np.float64), sys_.quads, models, e0, e1, mask=mask)
    out = rid.bias_force(S, E, torch.from_numpy(pos).cuda(), float(e0), float(e1),
                         conservative=True)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    bound = walker_bounds(got["eps"].astype(np.float64), ref["eps"], e0, e1)
    assert_walkers(got["F"], ref["F"], bound, f"length {length:g} {widths}")
    assert np.abs(got["eps"] / ref["eps"] - 1.0).max() <= FP32_TOL


def test_mask_set_changed_and_cleared(torch, rid):
    """Raw columns leave the packed weights with the mask and come back with
    it, before and after a training step."""
    n, widths, K, B = 19, [70, 64], 2, 21
    rng = np.random.default_rng(2)
    s = torch.from_numpy(ridgen.f32(rng.uniform(-2, 2, (B, n)))).cuda()
    params = ridgen.xavier_ensemble(2 * n, widths, K, 5, bias_std=0.1)
    masks = [(np.arange(n) % q != 0).astype(np.uint8) for q in (3, 18)] + [np.zeros(n, np.uint8), None]

    def outputs(E):
        return [o.cpu().numpy() for o in rid.model_dev(E, s)]

    E = rid.Ensemble(n, widths, K, params)
    for step in range(2):
        for m in masks + masks[::-1]:
            E.set_angular_mask(m)
            fresh = rid.Ensemble(n, widths, K, E.get_params())
            fresh.set_angular_mask(m)
            for a, b in zip(outputs(E), outputs(fresh)):
                assert np.array_equal(a, b)
        rid.mf_train_step(E, s, s, 1e-3)


@pytest.mark.parametrize("inf", [np.inf, -np.inf])
def test_infinite_raw_cvs_saturate(torch, rid, inf):
    """The same results as a value far past saturation, and other walkers as
    they were."""
    n, widths, K, B = 6, [70, 64], 2, 20
    mask = np.array([1, 0, 1, 1, 0, 1], np.uint8)
    s = ridgen.f32(np.random.default_rng(4).uniform(0.3, 1.5, (B, n)))
    E = _ensemble(rid, n, widths, K, ridgen.xavier_ensemble(2 * n, widths, K, 5, bias_std=0.1), mask,
                  False)

    def run(v):
        t = s.copy()
        if v is not None:
            t[7, 1] = v
        return [o.cpu().numpy() for o in rid.model_dev(E, torch.from_numpy(t).cuda())]

    plain, far, got = run(None), run(np.copysign(1e20, inf)), run(inf)
    keep = np.arange(B) != 7
    for p, f, g in zip(plain, far, got):
        assert np.array_equal(f, g) and np.isfinite(g).all() and np.array_equal(p[keep], g[keep])


@pytest.mark.parametrize("width,layers,resnet", [(64, 3, False), (256, 4, False), (300, 3, True)])
def test_same_bits_in_every_row_tile(torch, rid, width, layers, resnet):
    """Large calls (32 or 64 walkers a workgroup) and slices of them (16)."""
    n, K, B = 37, 4, 9000 if width == 64 else 4500
    s, mask, params, _ = _case(n, [width] * layers, K, B, 3.0, 12, resnet, every=3)
    E = _ensemble(rid, n, [width] * layers, K, params, mask, resnet)
    full = [o.cpu().numpy() for o in rid.model_dev(E, torch.from_numpy(s).cuda())]
    for lo, hi in ((0, 1), (37, 96), (B - 33, B)):
        part = rid.model_dev(E, torch.from_numpy(np.ascontiguousarray(s[lo:hi])).cuda())
        for a, b in zip(full, part):
            assert np.array_equal(a[lo:hi], b.cpu().numpy())
