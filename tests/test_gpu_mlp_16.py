"""The 16-bit MLP kernels at every padded width, against the FP64 oracle at the
edges of their tiles, and the same bits whatever row tile a walker lands in
and whether the encoding or positions come in.

Tolerances: those of the precision forms (gpu_common), per walker and member;
the free energy 1e-2 of the largest (the same roundings through the forward
sweep)."""
import numpy as np
import pytest

import ridgen
from oracle import rid_oracle as O
from tests.gpu_common import HALF_TOL

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


def _model(torch, rid, prec, n, widths, K, params, s):
    E = rid.Ensemble(n, widths, K, params, getattr(rid, "RID_" + prec.upper()))
    out = rid.model_dev(E, torch.from_numpy(s).cuda())
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


# each padded width below, at and above its edge, 5 and 6 hidden layers, inputs
# wider than the layers; 1, 15, 17, 33 and 65 walkers end in ragged tiles of
# 16, 32 and 64 rows; the large B take 32 rows and 64
@pytest.mark.parametrize("prec,n,widths,K,B", [
    ("fp16", 1, [1], 1, 1), ("bf16", 3, [63, 64], 2, 15), ("fp16", 38, [64] * 3, 8, 5000),
    ("bf16_all", 16, [65, 3, 40], 3, 17), ("fp16", 17, [128] * 6, 2, 33),
    ("bf16", 38, [120] * 4, 4, 1100), ("fp16", 38, [129] * 4, 4, 65),
    ("bf16_all", 33, [192] * 3, 5, 1030), ("bf16", 38, [193] * 4, 3, 1400),
    ("fp16", 48, [256] * 2, 4, 4100), ("fp16", 20, [257] * 4, 4, 1300),
    ("bf16", 18, [320] * 4, 4, 12), ("bf16_all", 18, [300] * 5, 4, 1300),
    ("fp16", 9, [321] * 4, 2, 31), ("bf16", 40, [384] * 3, 4, 4100),
    ("bf16_all", 60, [385] * 2, 2, 47), ("fp16", 64, [512] * 5, 2, 17),
    ("bf16", 120, [512] * 3, 4, 1030), ("fp16", 200, [130] * 2, 2, 40),
    ("bf16", 256, [512] * 2, 2, 35)])
def test_parity_at_tile_edges(torch, rid, prec, n, widths, K, B):
    rng = np.random.default_rng(n + B)
    s = ridgen.f32(rng.uniform(-np.pi, np.pi, (B, n)))
    params = ridgen.xavier_ensemble(2 * n, widths, K, 300 + n, bias_std=0.1)
    got = _model(torch, rid, prec, n, widths, K, params, s)
    sel = np.unique(np.concatenate([np.arange(min(B, 20)), np.arange(max(0, B - 40), B)]))
    A, g = O.ensemble_mean_force(ridgen.unpack_params(params, 2 * n, widths, K),
                                 s[sel].astype(np.float64))
    gg, Ag = got[3][sel], got[2][sel]
    # (the largest force of the members of a walker: a member's own may be tiny)
    err = np.abs(gg - g).max(axis=(1, 2)) / np.abs(g).max(axis=(1, 2))
    rms = np.linalg.norm(gg - g) / np.linalg.norm(g)
    errA = np.abs(Ag - A).max() / np.abs(A).max()
    print(f"{prec} n={n} {widths} K={K} B={B}: max {err.max():.2e} rms {rms:.2e} A {errA:.2e}",
          flush=True)
    tmax, trms = HALF_TOL[prec]
    assert err.max() <= tmax and rms <= trms and errA <= 1e-2


@pytest.mark.parametrize("prec,n,widths,K,B", [
    ("fp16", 38, [64] * 3, 4, 9000), ("bf16", 38, [100] * 3, 4, 2000),
    ("fp16", 38, [192] * 4, 4, 2000), ("bf16_all", 38, [256] * 4, 4, 4500),
    ("fp16", 38, [256] * 4, 4, 2001), ("bf16", 18, [300] * 4, 4, 4200),
    ("fp16", 38, [384] * 3, 4, 4100), ("bf16", 38, [512] * 3, 4, 4100),
    ("fp16", 38, [200] * 6, 4, 2000)])
def test_same_bits_in_every_row_tile(torch, rid, prec, n, widths, K, B):
    """A large call (32 or 64 rows a workgroup) and calls on its slices (16
    rows, other places in the tile) give the same bits."""
    rng = np.random.default_rng(5)
    s = ridgen.f32(rng.uniform(-np.pi, np.pi, (B, n)))
    params = ridgen.xavier_ensemble(2 * n, widths, K, 77, bias_std=0.1)
    full = _model(torch, rid, prec, n, widths, K, params, s)
    for lo, hi in ((0, 1), (37, 96), (700, 1300), (B - 33, B)):
        part = _model(torch, rid, prec, n, widths, K, params, np.ascontiguousarray(s[lo:hi]))
        for a, b in zip(full, part):
            assert np.array_equal(a[lo:hi], b)


@pytest.mark.parametrize("width,K", [(64, 3), (300, 4), (512, 2)])
def test_positions_in_every_row_tile(torch, rid, width, K):
    """The bias path: torsions gathered by waves that do not divide the rows
    evenly, in tiles of 16 and more walkers, the same bits."""
    sys_ = ridgen.system_peptide20()
    B = 1100
    pos = ridgen.f32(ridgen.chain_coords(sys_, B, 3))
    widths = [width] * 3
    params = ridgen.xavier_ensemble(2 * sys_.n_cv, widths, K, 9, bias_std=0.1)
    S = rid.System(sys_.n_atoms, sys_.quads)
    E = rid.Ensemble(sys_.n_cv, widths, K, params, rid.RID_FP16)
    dev = torch.from_numpy(pos).cuda()

    def run(p):
        out = rid.bias_force(S, E, p.contiguous(), 0.5, 2.0)
        torch.cuda.synchronize()
        return [out[q].cpu().numpy() for q in ("F", "E", "eps", "sigma", "flags")]

    full = run(dev)
    for lo, hi in ((0, 1), (100, 137), (B - 20, B)):
        for a, b in zip(full, run(dev[lo:hi])):
            assert np.array_equal(a[lo:hi], b)


@pytest.mark.parametrize("res,prec,width,K", [
    (2, "fp32", 64, 4), (2, "fp16", 100, 3), (10, "fp16", 128, 4), (10, "bf16", 300, 4),
    (10, "fp32", 300, 4), (20, "fp32", 192, 3), (20, "fp32", 256, 4), (16, "bf16_all", 384, 4),
    (13, "fp16", 512, 8), (10, "fp32", 512, 4)])
def test_torsions_in_the_kernel_and_encoded_first(torch, rid, res, prec, width, K):
    """Calls of one round of workgroups with few torsions a wave compute them
    in the MLP kernel, larger ones encode first: the same bits."""
    sys_ = ridgen.chain_system(res, 12)
    n, B, widths = sys_.n_cv, 16 * (256 // K + 2), [width] * 3
    pos = torch.from_numpy(ridgen.f32(ridgen.chain_coords(sys_, B, 4))).cuda()
    S = rid.System(sys_.n_atoms, sys_.quads)
    E = rid.Ensemble(n, widths, K, ridgen.xavier_ensemble(2 * n, widths, K, 6, bias_std=0.1),
                     getattr(rid, "RID_" + prec.upper()))

    def run(p):
        out = rid.bias_force(S, E, p.contiguous(), 0.5, 2.0)
        torch.cuda.synchronize()
        return [out[q].cpu().numpy() for q in ("F", "E", "eps", "sigma", "flags")]

    full = run(pos)
    for lo, hi in ((0, 1), (100, 137), (B - 300, B)):
        for a, b in zip(full, run(pos[lo:hi])):
            assert np.array_equal(a[lo:hi], b)
