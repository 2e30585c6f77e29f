"""A weight packing that could not be launched is tried again: the call reports
the error, and the next one packs before it evaluates, so no call evaluates
weights older than the last training step.  On the CPU, the HIP runtime
replaced (hip_stub)."""
import pytest

from tests import hip_stub


@pytest.mark.parametrize("prec,kernel", [("RID_FP32", "pack_split_kernel"),
                                         ("RID_FP16", "pack_kernel")])
@pytest.mark.parametrize("call", [
    "L.rid_model_dev(E, ptr(s), B, ptr(eps), None, None, None, None)",
    "L.rid_bias_force(S, E, ptr(pos), B, 0.5, 2.0, ptr(out), None, None, None, None, None)",
    "L.rid_mcmc_run(E, ptr(s), B, 1, 0, 1.0, 0.1, 1, 0, 1, 8, ptr(hist), None, None, None)"])
def test_failed_packing_is_repeated(tmp_path, prec, kernel, call):
    hip_stub.run(tmp_path, f"""
        spec = ridgen.chain_system(4, 12)
        n, K, B = spec.n_cv, 2, 20
        S, E = system(spec), ensemble(n, [64, 64], K, rid.{prec})
        s = np.zeros((B, n), np.float32)
        pos = np.zeros((B, spec.n_atoms, 3), np.float32)
        eps, out, hist = np.zeros(B, np.float32), np.zeros_like(pos), np.zeros((n, 8), np.uint32)
        assert {call} == 0
        assert not any({kernel!r} in k for k in launched())
        assert L.rid_mf_train_step(E, ptr(s), ptr(s), B, 1e-3, None, None) == 0
        launched()
        stub.stub_fail_next_launch({kernel!r}.encode())
        assert {call} == rid.RID_EDEVICE
        launched()
        assert {call} == 0
        assert any({kernel!r} in k for k in launched()), "evaluated without packing"
        assert {call} == 0
        assert not any({kernel!r} in k for k in launched())
        """)
