"""Device memory near a context's budget: what decides between a resident ensemble, one
paged member set and two, and what a call leaves behind."""
import numpy as np
import pytest

from paper_2604_02755_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_estimate_counts_the_partial_sums(nlth_mod):
    """A budget short of the ensemble by half its partial-sum buffer (17,152 rows of 64
    doubles): two member sets, as for every ensemble that does not fit."""
    members = 64
    mesh = I.box_mesh(12, 12, 8, 1.0, I.two_layer(2.0), 6)
    rng = np.random.default_rng(4)
    prob = I.make_problem(members, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], n_springs=12, n_steps=2,
                          input_acc=40.0 * rng.standard_normal((members, 2, 3)))

    def run(budget):
        print("budget case", budget, flush=True)
        ctx = nlth_mod.Context(0, hbm_budget=budget, use_torch_stream=False)
        try:
            ens = ctx.ensemble(ctx.mesh(mesh), mesh, prob)
            ens.step(2)
            st, out = ens.stats(), ens.read()
            ens.close()
            return st, out
        finally:
            ctx.close()

    whole, ref = run(0)
    assert whole["member_sets"] == 1 and not whole["paged"]
    st, out = run(whole["device_bytes"] - 17152 * members * 8 // 2)
    assert st["paged"] and st["member_sets"] == 2
    assert np.abs(ref["vel"]).max() > 0
    assert np.linalg.norm(out["vel"] - ref["vel"]) < 1e-7 * np.linalg.norm(ref["vel"])
