"""Where the chunks of CG iterations that are issued together end changes no result."""
import numpy as np
import pytest

from paper_2604_02755_amd import inputs as I

pytestmark = pytest.mark.gpu


def _problem(members, n_steps, **kw):
    rng = np.random.default_rng(members)
    acc = 40.0 * rng.standard_normal((members, n_steps, 3))
    prob = I.make_problem(members, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], gamma_ref=rng.uniform(5e-4, 2e-3, members),
                          n_springs=12, n_steps=n_steps, input_acc=acc, **kw)
    prob.vs = np.ascontiguousarray(prob.vs * np.exp(0.2 * rng.standard_normal(prob.vs.shape)))
    return prob


# (12, 12, 9) with 2 members: about 93 blocks of the update kernel and 460 of the
# operator, so the p update joins the operator within a chunk and the beta stage sums
# more rows than a wavefront of either kernel has lanes for a member
@pytest.mark.parametrize("members,dims", [(1, (12, 12, 9)), (2, (12, 12, 9)), (2, (4, 3, 3)), (4, (12, 12, 9))])
@pytest.mark.parametrize("precision", [0, 1])
def test_chunk_lengths_give_the_same_bits(nlth_mod, members, dims, precision):
    mesh = I.box_mesh(*dims, 1.0, I.two_layer(2.0), 4)
    prob = _problem(members, 4, cg_tol=1e-10, precision=precision)
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        mh = ctx.mesh(mesh)

        def run(p, check_every):
            print("chunk case", members, dims, precision, check_every, flush=True)
            ens = ctx.ensemble(mh, mesh, p)
            try:
                ens.set_tuning(check_every=check_every)
                ens.step(p.n_steps)
                return ens.read()
            finally:
                ens.close()

        ref = run(prob, 1)
        assert np.abs(ref["vel"]).max() > 0
        for ce in (3, 4, 16):
            got = run(prob, ce)
            assert np.array_equal(got["iters"], ref["iters"])
            assert np.abs(got["vel"] - ref["vel"]).max() == 0.0
        if members > 1:  # the other member at rest: its solves end at once, the chunks elsewhere
            still = _problem(members, 4, cg_tol=1e-10, precision=precision)
            still.input_acc[1:] = 0.0
            assert np.abs(run(still, 8)["vel"][0] - ref["vel"][0]).max() == 0.0
    finally:
        ctx.close()
