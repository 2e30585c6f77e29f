"""What a call of rid_bias_force allocated serves every later call of the same
size or less, whatever route that takes (a call under graph capture cannot
allocate): one ensemble, a system whose torsions the MLP kernel gathers itself
and one with more torsion atoms, whose CVs are encoded first.  On the CPU, the
HIP runtime replaced (hip_stub)."""
import pytest

from tests import hip_stub


@pytest.mark.parametrize("prec,width,res", [("RID_FP32", 256, 16), ("RID_FP16", 128, 6)])
def test_bias_force_allocates_for_both_routes(tmp_path, prec, width, res):
    hip_stub.run(tmp_path, f"""
        few = ridgen.chain_system({res}, 12)          # 2 res - 2 torsions of 3 res atoms
        # the same number of torsions, each of four atoms of its own
        class Many: pass
        many = Many()
        many.n_cv, many.n_atoms = few.n_cv, 4 * few.n_cv
        many.quads = np.arange(4 * few.n_cv, dtype=np.int32).reshape(-1, 4)
        n, K, B = few.n_cv, 4, 100
        E = ensemble(n, [{width}] * 3, K, rid.{prec})
        def call(spec, S, b):
            pos = np.zeros((b, spec.n_atoms, 3), np.float32)
            out = np.zeros_like(pos)
            r = L.rid_bias_force(S, E, ptr(pos), b, 0.5, 2.0, ptr(out), None, None, None, None, None)
            return r, launched()
        Sf, Sm = system(few), system(many)
        r, k = call(few, Sf, B)
        assert r == 0 and not any("cv_eval" in q for q in k), k
        stub.stub_fail_allocations(1)
        for spec, S in ((few, Sf), (many, Sm), (many, Sm)):
            for b in (B, 1):
                r, k = call(spec, S, b)
                assert r == 0, (spec is few, b, L.rid_last_error())
        assert any("cv_eval" in q for q in k), k
        """)
