"""Iterations that are issued before the members' flags are looked at: a hard solve
does not make the next one as long."""
import numpy as np
import pytest

from paper_2604_02755_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("members", [2, 5])
def test_solve_after_a_member_failed(nlth_mod, members):
    mesh = I.box_mesh(6, 5, 4, 1.0, I.two_layer(2.0), 2)
    rng = np.random.default_rng(2)
    prob = I.make_problem(members, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], n_springs=12, n_steps=4,
                          input_acc=40.0 * rng.standard_normal((members, 4, 3)), cg_tol=1e-10, cg_maxit=600)
    prob.nu[-1] = 0.4999  # nearly incompressible: more than 1,000 iterations where the others take 60
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        ens = ctx.ensemble(ctx.mesh(mesh), mesh, prob)
        ens.set_profile(True)
        issued = []
        for step in range(3):
            print("failed member case", members, step, flush=True)
            ens.reset_stats()
            with pytest.raises(nlth_mod.NlthError) as e:
                ens.step(1)
            assert e.value.code == nlth_mod.NLTH_ENOCONV
            issued.append(ens.stats()["n_ebe64"])
        out = ens.read()
        ens.close()
    finally:
        ctx.close()
    took = out["iters"][:, :, 0]
    print(issued, took[:, :3].tolist(), flush=True)
    assert out["status"].tolist() == [0] * (members - 1) + [nlth_mod.NLTH_ENOCONV] and took[-1, 0] == 600
    for step in (1, 2):  # right-hand side, initial residual and K du, and two chunks of 8
        assert 0 < took[:-1, step].max() < 100 and issued[step] <= took[:-1, step].max() + 3 + 16


def test_wide_inner_solve_after_a_long_one(nlth_mod):
    """64 slots, all members alike, a check after every iteration: the inner solves of a
    step at a loose tolerance issue what they take, also after one at a tight tolerance."""
    mesh = I.box_mesh(6, 5, 4, 1.0, I.two_layer(2.0), 2)
    acc = np.tile(40.0 * np.random.default_rng(2).standard_normal((1, 2, 3)), (64, 1, 1))
    prob = I.make_problem(64, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], n_springs=12, n_steps=2, input_acc=acc,
                          precision=1)
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        ens = ctx.ensemble(ctx.mesh(mesh), mesh, prob)
        ens.set_profile(True)
        issued = []
        for step, tol in enumerate((1e-5, 0.5)):
            print("inner issue case", step, tol, flush=True)
            ens.set_tuning(check_every=1, inner_tol=tol)
            ens.reset_stats()
            ens.step(1)
            issued.append(ens.stats()["n_ebe32"])
        it = ens.read()["iters"]
        ens.close()
    finally:
        ctx.close()
    print(issued, it[:4].tolist(), flush=True)
    assert (it == it[:1]).all() and it[0, 0, 1] > 20 * it[0, 0, 0] and it[0, 1, 1] < 6 * it[0, 1, 0]
    assert issued == it[0, :, 1].tolist()
