"""The allocation-free application stages its D rows with 16-byte loads where the
buffer allows: buffers that start 8 bytes off, meshes whose last cluster is
partly filled, and every operator give the same bits as the aligned call."""
import numpy as np
import pytest

from paper_2604_02755_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 2, 2), (5, 4, 3), (9, 8, 7)])
def test_offset_buffers_give_the_same_bits(nlth_mod, dims):
    import torch
    ctx = nlth_mod.Context(0, use_torch_stream=False)
    try:
        mesh, prob = I.config(0, n_steps=1, mesh_dims=dims)
        mh = ctx.mesh(mesh)
        rng = np.random.default_rng(sum(dims))
        a = rng.normal(size=(mesh.n_tets, 4, 6, 6))
        full = a @ a.transpose(0, 1, 3, 2) + 10 * np.eye(6)
        D = full[..., np.triu_indices(6)[0], np.triu_indices(6)[1]].reshape(-1)
        h, x = rng.uniform(0, 0.2, mesh.n_tets), rng.normal(size=mesh.n_dof)

        def buf(v, off):
            t = torch.zeros(v.size + 2, dtype=torch.float64, device="cuda")
            t[off:off + v.size] = torch.from_numpy(v).cuda()
            return t, t.data_ptr() + 8 * off

        for which in (0, 1, 2):
            got = []
            for off in (0, 1):
                keep = [buf(v, off) for v in (D, h, x)]
                y, yp = buf(np.full(mesh.n_dof, np.nan), off)
                torch.cuda.synchronize()
                print("alignment case", dims, which, off, flush=True)
                nlth_mod.nlth_apply_operator_noalloc(ctx.h, mh, prob, which, keep[0][1], keep[1][1], keep[2][1], yp)
                torch.cuda.synchronize()
                got.append(y[off:off + mesh.n_dof].cpu().numpy())
            ref = ctx.apply_operator(mh, prob, which, 0, D.reshape(-1, 4, 21), h, x)
            assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], ref) and np.abs(ref).max() > 0
    finally:
        ctx.close()
