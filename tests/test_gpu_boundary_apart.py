"""FP32 operator of 256 slots and about 30,000 cluster blocks, whose dashpot rows are a
launch of their own, against the colour path, at the nodes that have such rows (CG at
1e-12: the bar of the mixed parity runs, 1e-9)."""
import numpy as np
import pytest

from paper_2604_02755_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_dashpot_rows_of_their_own_match_the_colour_path(nlth_mod):
    members = 250  # lanes left empty in the last group
    mesh = I.box_mesh(30, 24, 16, 1.0, I.two_layer(4.0), 6)
    mesh.recv = np.unique(mesh.bface6).astype(np.int32)  # the boundary nodes: the base moves in the first step
    rng = np.random.default_rng(9)
    prob = I.make_problem(members, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], gamma_ref=rng.uniform(5e-4, 2e-3, members),
                          n_springs=12, n_steps=1, input_acc=40.0 * rng.standard_normal((members, 1, 3)), cg_tol=1e-12,
                          precision=1, inner_dtype=2)
    prob.vs = np.ascontiguousarray(prob.vs * np.exp(0.2 * rng.standard_normal(prob.vs.shape)))
    prob.dirs, prob.weights = np.ascontiguousarray(prob.dirs[:2]), np.full(2, 2.5)  # (a small law state)
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        mh = ctx.mesh(mesh)
        info = nlth_mod.nlth_mesh_query(ctx.h, mh, mesh.n_tets)[0]
        assert info.n_clusters * 4 > 28672
        got = []
        for scatter in (-1, 1):
            print("dashpot rows case", scatter, flush=True)
            ens = ctx.ensemble(mh, mesh, prob)
            ens.set_tuning(scatter=scatter)
            ens.step(1)
            got.append(ens.read())
            ens.close()
    finally:
        ctx.close()
    a, b = got
    print(a["iters"][:3, 0].tolist(), b["iters"][:3, 0].tolist(), flush=True)
    assert np.all(a["status"] == 0) and np.all(b["status"] == 0) and np.abs(b["vel"]).max() > 0
    assert np.linalg.norm(a["vel"] - b["vel"]) < 1e-9 * np.linalg.norm(b["vel"])
