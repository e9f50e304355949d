"""The column preconditioner of the global solve over the heights and orders at which
its tiles change (16 levels a tile, up to 130 levels; orders 2 to 6).  On a mesh of
1e14 m the horizontal terms of the global operator are below 1e-10 of the vertical
ones (sound speed times alpha over the node distance), so it is the column operator of
each column, and the preconditioned solve to 1e-9 has to end after one Arnoldi step."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [(2, 2), (2, 7), (3, 5), (5, 3), (4, 4), (3, 11), (4, 10), (6, 8), (5, 13), (2, 40), (4, 24), (3, 37),
         (4, 31), (3, 43)]   # n_z = 5, 15, 16, 16, 17, 34, 41, 49, 66, 81, 97, 112, 125, 130


@pytest.mark.parametrize("N,nelz", CASES)
def test_column_preconditioner(N, nelz):
    import torch
    from paper_2504_08157_amd import nhsem
    mesh = W.MeshSpec((5, 3, nelz), N, W.uniform_edges(0, 1e14, 5), W.uniform_edges(0, 1e14, 3),
                      W.stretched_edges(0, 12e3, nelz, seed=3), (True, True))
    ctx = nhsem.Context(mesh, W.Physics())
    x, y, z = ctx.nh_lattice_coords()
    ctx.nh_set_reference(*W.constant_n_reference(z))
    rng = np.random.default_rng(N * nelz)
    # every column of its own, w not zero at the walls
    b = rng.normal(size=(5, mesh.U)) * np.array([1e-3, 1.0, 1.0, 1.0, 1.0])[:, None]
    b = torch.from_numpy(b).cuda()
    alpha = 1.5
    got, st = ctx.nh_global_solve(alpha, b, x0=torch.zeros_like(b), restart=10, rtol=1e-9, precondition=True)
    assert st.iters_total == 1 and st.not_converged == 0, st.iters_total
    r = b - (got - alpha * ctx.nh_l3_apply(got))
    assert r.norm() <= 2e-9 * b.norm()
