"""A column solve whose step counts go to the caller's array does not write the
attached HEVI workspace, which a caller may lend to several contexts on streams of
their own; its statistics and the diagnostics of the same context keep apart."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nel,restart", [((3, 2, 4), 10), ((3, 2, 4), 20), ((2, 2, 18), 10),
                                         ((16, 8, 3), 10), ((16, 9, 3), 10)])
def test_column_solve_leaves_the_workspace(nel, restart):
    import torch
    from paper_2504_08157_amd import nhsem
    mesh = W.MeshSpec(nel, 4, W.uniform_edges(0, 5e5, nel[0]), W.uniform_edges(0, 4e5, nel[1]),
                      W.uniform_edges(0, 12e3, nel[2]), (True, True))
    ctx = nhsem.Context(mesh, W.Physics())
    c = ctx.nh_lattice_coords()
    ctx.nh_set_reference(*W.constant_n_reference(c[2]))
    ctx.nh_hevi_attach()
    rng = np.random.default_rng(nel[2])
    scale = np.array([1e-3, 1.0, 1.0, 1.0, 1.0])[:, None]
    b = torch.from_numpy(rng.normal(size=(5, mesh.U)) * scale).cuda()
    ctx.nh_set_state(b)
    diag = ctx.nh_diagnostics()
    it = torch.zeros(len(c[0]) * len(c[1]), dtype=torch.int32, device="cuda")
    ctx.hws.fill_(0xA5)
    _, st = ctx.nh_column_solve(1.5, b, restart=restart, max_restarts=60, rtol=1e-9, iters=it)
    assert st.iters_total == int(it.sum()) > 0 and st.iters_max == int(it.max())
    assert bool((ctx.hws == 0xA5).all())
    np.testing.assert_array_equal(np.asarray(ctx.nh_diagnostics()), np.asarray(diag))
