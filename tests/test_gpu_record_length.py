"""What a run does at a step does not depend on samples that come later: the same
first steps of a longer record, and a request served alone in its batch (whose record
is padded), give the bits of the short run."""
import numpy as np
import pytest

from paper_2604_02755_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_steps", [5, 64, 70])
@pytest.mark.parametrize("precision", [0, 1])
def test_longer_record_gives_the_same_first_steps(nlth_mod, precision, n_steps):
    mesh = I.box_mesh(3, 2, 2, 1.0, I.two_layer(1.0), 2)
    rng = np.random.default_rng(n_steps)
    acc = 40.0 * rng.standard_normal((2, n_steps + 700, 3))
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        mh = ctx.mesh(mesh)
        got = []
        for record in (n_steps, n_steps + 1, n_steps + 700):
            prob = I.make_problem(2, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], n_springs=12, n_steps=record,
                                  input_acc=acc[:, :record], cg_tol=1e-10, precision=precision)
            print("record case", precision, n_steps, record, flush=True)
            ens = ctx.ensemble(mh, mesh, prob)
            ens.step(n_steps)
            got.append(ens.read()["vel"][:, :n_steps])
            ens.close()
        prob = I.make_problem(1, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], n_springs=12, n_steps=n_steps,
                              input_acc=acc[:1, :n_steps], cg_tol=1e-10, precision=precision)
        ticket, served = ctx.submit(mh, mesh, prob)
        assert ctx.wait(ticket, 60.0) == 0
        ctx.release(ticket)
        alone = ctx.solve_as_served(mh, mesh, prob)
    finally:
        ctx.close()
    assert np.abs(got[0]).max() > 0
    assert np.abs(got[1] - got[0]).max() == 0.0 and np.abs(got[2] - got[0]).max() == 0.0
    assert np.abs(served["vel"] - alone["vel"]).max() == 0.0


def test_incident_velocity_over_a_long_record(nlth_mod, oracle_lib):
    """A record of 1,000 samples (fifteen times what a wavefront holds, and a remainder),
    member by member against the oracle."""
    mesh = I.box_mesh(2, 2, 1, 1.0, I.two_layer(1.0), 1)
    acc = I.member_waves(0, range(3), 1000, 1e-3) * 5.0
    prob = I.make_problem(3, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], n_springs=12, n_steps=1000, input_acc=acc,
                          cg_tol=1e-12)
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        print("long record case", flush=True)
        out = ctx.solve(ctx.mesh(mesh), mesh, prob)
    finally:
        ctx.close()
    for m in range(3):
        ref = oracle_lib.run(mesh, prob, member=m)
        err = oracle_lib.rel_l2(out["vel"][m], ref["vel"])
        print("  member", m, "rel L2 vs oracle", err, flush=True)
        assert np.abs(ref["vel"]).max() > 0 and err < 1e-9
