"""Law of many springs on a mesh whose chunks are small and whose whole is not: the
paged run sums the springs in the resident run's order (same kernels, same bits)."""
import numpy as np
import pytest

from paper_2604_02755_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,members", [((12, 8, 8), 4), ((6, 5, 4), 4)])  # 73,728 and 11,520 point-members
@pytest.mark.parametrize("depth", [1, 3])
def test_paged_law_gives_the_resident_bits(nlth_mod, dims, members, depth):
    mesh = I.box_mesh(*dims, 1.0, I.two_layer(2.0), 4)
    mesh.recv = np.unique(mesh.bface6[::5]).astype(np.int32)  # boundary nodes: the base moves at once
    rng = np.random.default_rng(3)
    prob = I.make_problem(members, I.CFG0_LAYERS["vs"], I.CFG0_LAYERS["rho"], gamma_ref=rng.uniform(2e-4, 5e-4, members),
                          n_springs=150, n_steps=4, input_acc=60.0 * rng.standard_normal((members, 4, 3)), cg_tol=1e-10,
                          masing_depth=depth)
    pick = np.linspace(0, 149, 60).round().astype(int)
    prob.dirs, prob.weights = np.ascontiguousarray(prob.dirs[pick]), np.full(60, 5.0 / 60)
    got = []
    for budget in (0, None):
        if budget is None:  # what the resident run took, less half its law state
            budget = st["device_bytes"] - mesh.n_tets * 4 * 60 * 4 * 36 // 2
        print("paged parts case", dims, depth, budget, flush=True)
        ctx = nlth_mod.Context(0, hbm_budget=budget, use_torch_stream=False, paging_sets=1)
        try:
            ens = ctx.ensemble(ctx.mesh(mesh), mesh, prob)
            ens.step(prob.n_steps)
            st = ens.stats()
            got.append(ens.read())
            ens.close()
        finally:
            ctx.close()
        assert bool(st["paged"]) == (len(got) == 2)
    assert np.abs(got[0]["vel"]).max() > 0
    assert np.abs(got[0]["vel"] - got[1]["vel"]).max() == 0.0
