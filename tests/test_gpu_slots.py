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


@pytest.mark.parametrize("members,dims", [(1, (5, 3, 3)), (2, (9, 8, 7)), (3, (8, 8, 8)), (8, (16, 16, 17)), (16, (10, 8, 8)),
                                          (32, (10, 8, 8)), (70, (6, 5, 4))])
@pytest.mark.parametrize("precision", [0, 1])
def test_iterations_match_the_colour_path(nlth_mod, members, dims, precision):
    """The stages of a CG iteration formed inside the update kernels (few sums, and
    folded sums from 16 slots on), launched (8 slots, 26,112 tets), and the
    diagonal by clusters, against the colour path with its separate stages and one
    diagonal launch per colour: as many iterations (one more or less where a
    residual lies at the tolerance within rounding), the same velocities, and the
    same member status when the iteration limit stops the solve."""
    mesh = I.box_mesh(*dims, 1.0, I.two_layer(1.0), 2)
    rng = np.random.default_rng(members)
    acc = 40.0 * rng.standard_normal((members, 3, 3))
    prob = I.make_problem(members, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], gamma_ref=rng.uniform(5e-4, 2e-3, members),
                          n_springs=12, n_steps=3, input_acc=acc, cg_tol=1e-12, precision=precision)
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        mh = ctx.mesh(mesh)
        for maxit in (2000, 2):
            prob.cg_maxit = maxit
            got = []
            for scatter in (-1, 1):
                print("stages case", members, dims, precision, maxit, scatter, flush=True)
                ens = ctx.ensemble(mh, mesh, prob)
                try:
                    if scatter == 1:
                        ens.set_tuning(scatter=1)
                    try:
                        ens.step(prob.n_steps)
                    except nlth_mod.NlthError as e:
                        assert maxit == 2 and e.code == nlth_mod.NLTH_ENOCONV
                    got.append(ens.read())
                finally:
                    ens.close()
            a, b = got
            assert np.array_equal(a["status"], b["status"])
            if maxit == 2:
                assert np.all(a["status"] == nlth_mod.NLTH_ENOCONV) and np.array_equal(a["iters"][..., 0], b["iters"][..., 0])
                continue
            assert np.all(a["status"] == 0) and np.abs(b["vel"]).max() > 0
            print("  iterations", a["iters"][0, :, 0], b["iters"][0, :, 0], flush=True)
            assert np.abs(a["iters"][..., 0] - b["iters"][..., 0]).max() <= 1
            assert np.linalg.norm(a["vel"] - b["vel"]) < 1e-9 * np.linalg.norm(b["vel"])
    finally:
        ctx.close()


@pytest.mark.parametrize("depth", [1, 3])
@pytest.mark.parametrize("springs,dims,members", [(17, (5, 3, 3), 2), (150, (5, 3, 3), 1), (37, (8, 8, 8), 2),
                                                  (150, (8, 6, 4), 16), (18, (8, 8, 8), 8)])
def test_springs_in_parts_match_oracle(nlth_mod, oracle_lib, springs, dims, members, depth):
    """The law with more springs than the LDS form takes: 8 wavefronts a block
    sharing them (up to 16,384 element-point-members), 4 (up to 65,536), and none,
    with spring counts that the parts do not divide."""
    mesh = I.box_mesh(*dims, 1.0, I.two_layer(1.0), 2)
    rng = np.random.default_rng(springs)
    acc = 60.0 * rng.standard_normal((members, 5, 3))
    prob = I.make_problem(members, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], gamma_ref=rng.uniform(2e-4, 5e-4, members),
                          n_springs=150, n_steps=5, input_acc=acc, cg_tol=1e-12, masing_depth=depth)
    pick = np.linspace(0, 149, springs).round().astype(int)
    prob.dirs, prob.weights = np.ascontiguousarray(prob.dirs[pick]), np.full(springs, 5.0 / springs)
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        mh = ctx.mesh(mesh)
        print("springs case", springs, dims, members, depth, flush=True)
        out = ctx.solve(mh, mesh, prob)
    finally:
        ctx.close()
    assert out["rc"] == 0
    ref = oracle_lib.run(mesh, prob, member=members - 1)
    err = oracle_lib.rel_l2(out["vel"][members - 1], ref["vel"])
    print("  rel L2 vs oracle", err, flush=True)
    assert np.abs(ref["vel"]).max() > 0 and err < 1e-9
