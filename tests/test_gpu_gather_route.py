"""Torsions computed in the MLP kernel at shapes where that route is taken
(counted by the CV kernel's launches): waves that do not divide the 16 walkers
of a tile evenly (widths 192, 320 and 384), one walker, ragged tiles, FP32 and
16-bit; the same bits as the calls that encode the CVs first."""
import numpy as np
import pytest

import ridgen

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


@pytest.mark.parametrize("res,prec,width,K", [
    (4, "fp16", 64, 4), (6, "fp16", 128, 4), (9, "bf16", 192, 3), (10, "fp16", 300, 4),
    (12, "bf16_all", 384, 4), (9, "bf16", 512, 3), (5, "fp32", 64, 4), (9, "fp32", 128, 2),
    (12, "fp32", 180, 3), (10, "fp32", 300, 4), (15, "fp32", 384, 5), (20, "fp32", 512, 4)])
def test_gathered_and_encoded_first(torch, rid, res, prec, width, K):
    sys_ = ridgen.chain_system(res, 12)
    n, B, widths = sys_.n_cv, 16 * (256 // K + 2), [width] * 3
    pos = torch.from_numpy(ridgen.f32(ridgen.chain_coords(sys_, B, 4))).cuda()
    S = rid.System(sys_.n_atoms, sys_.quads)
    E = rid.Ensemble(n, widths, K, ridgen.xavier_ensemble(2 * n, widths, K, 6, bias_std=0.1),
                     getattr(rid, "RID_" + prec.upper()))

    def run(p):
        rid.profile_enable(True)
        out = rid.bias_force(S, E, p.contiguous(), 0.5, 2.0)
        torch.cuda.synchronize()
        encoded = rid.profile_read(rid.PROF_CV)[1]
        rid.profile_enable(False)
        return [out[q].cpu().numpy() for q in ("F", "E", "eps", "sigma", "flags")], encoded

    full, encoded = run(pos)
    assert encoded == 1
    for lo, hi in ((0, 1), (100, 137), (B - 300 if B > 300 else 0, B - 40)):
        part, encoded = run(pos[lo:hi])
        assert encoded == 0, "the MLP kernel was to compute the torsions"
        for a, b in zip(full, part):
            assert np.array_equal(a[lo:hi], b)
