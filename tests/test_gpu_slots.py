"""Ensembles of few member slots (1 to 32): the operator's form for each slot
count, with member counts that leave lanes empty and boxes whose elements leave
a cluster and a pass partly filled, against the oracle.  CG at 1e-12 and FP64
sums: the bars are those of the FP64 and mixed parity runs (1e-9)."""
import numpy as np
import pytest

from paper_2604_02755_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("members", [1, 2, 3, 7, 13, 32])
@pytest.mark.parametrize("precision,inner", [(0, 0), (1, 0), (1, 1), (1, 2)])
def test_slot_counts_match_oracle(nlth_mod, oracle_lib, members, precision, inner):
    dims = (3, 2, 2) if members > 8 else (5, 3, 3)  # 72 and 270 tets: part clusters of 64 and of 12
    mesh = I.box_mesh(*dims, 1.0, I.two_layer(1.0), 2)
    rng = np.random.default_rng(members)
    acc = 40.0 * rng.standard_normal((members, 6, 3))
    prob = I.make_problem(members, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], gamma_ref=rng.uniform(5e-4, 2e-3, members),
                          n_springs=12, n_steps=6, input_acc=acc, cg_tol=1e-12, precision=precision, inner_dtype=inner)
    prob.vs = np.ascontiguousarray(prob.vs * np.exp(0.2 * rng.standard_normal(prob.vs.shape)))
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        mh = ctx.mesh(mesh)
        print("slots case", members, precision, inner, flush=True)
        out = ctx.solve(mh, mesh, prob)
    finally:
        ctx.close()
    assert out["rc"] == 0
    for m in {0, members // 2, members - 1}:
        ref = oracle_lib.run(mesh, prob, member=m)
        err = oracle_lib.rel_l2(out["vel"][m], ref["vel"])
        print("  member", m, "rel L2 vs oracle", err, flush=True)
        assert np.abs(ref["vel"]).max() > 0 and err < 1e-9
