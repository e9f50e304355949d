"""Statistics of the column solves: summed on the GPU with a HEVI workspace attached, on
the host without one; both against the per-column counts, on few and many columns, with
columns that miss rtol."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nel,max_restarts", [((2, 2, 3), 20), ((19, 13, 4), 20), ((19, 13, 4), 0), ((70, 60, 2), 20)])
def test_solve_stats(nel, max_restarts):
    import torch
    from paper_2504_08157_amd import nhsem
    mesh = W.MeshSpec(nel, 4, W.uniform_edges(0, 5e5, nel[0]), W.uniform_edges(0, 4e5, nel[1]),
                      W.uniform_edges(0, 12e3, nel[2]), (True, True))
    ctx = nhsem.Context(mesh, W.Physics())
    c = ctx.nh_lattice_coords()
    ctx.nh_set_reference(*W.constant_n_reference(c[2]))
    rng = np.random.default_rng(nel[0])
    scale = np.array([1e-3, 1.0, 1.0, 1.0, 1.0])[:, None]
    b = torch.from_numpy(rng.normal(size=(5, mesh.U)) * scale).cuda()
    ncol = len(c[0]) * len(c[1])
    got = []
    for attached in (False, True):
        if attached:
            ctx.nh_hevi_attach()
        it = torch.full((ncol,), 12345, dtype=torch.int32, device="cuda")
        # restart 4 and no restart: some columns miss rtol
        _, st = ctx.nh_column_solve(1.5, b, restart=4, max_restarts=max_restarts, rtol=1e-9, iters=it, check=False)
        v = it.cpu().numpy().astype(np.int64)
        steps = np.where(v >= 0, v, -v - 1)
        want = (ncol, 1, int(steps.sum()), int(steps.max()), int((v < 0).sum()))
        assert (st.columns, st.solves, st.iters_total, st.iters_max, st.not_converged) == want
        got.append(want)
    assert got[0] == got[1] and (max_restarts > 0 or got[0][4] > 0)
