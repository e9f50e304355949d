"""Columns whose right-hand side holds an infinity or a NaN: reported as not converged,
without a value in any other column's solution changed."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu


# columns of 1 to 17 elements, the walls and the levels beside them
@pytest.mark.parametrize("field,level", [(0, 0), (0, 1), (0, -1), (3, 0), (3, 1), (4, 0), (4, 2), (4, -1)])
@pytest.mark.parametrize("N,nelz", [(2, 1), (2, 16), (3, 5), (4, 3), (4, 16), (5, 10), (6, 2), (6, 10), (4, 17)])
@pytest.mark.parametrize("restart,schur", [(10, True), (10, False), (20, False)])
def test_nonfinite_column(N, nelz, restart, schur, field, level):
    import torch
    from paper_2504_08157_amd import nhsem
    H = 15e3
    mesh = W.MeshSpec((2, 2, nelz), N, W.uniform_edges(0, 20e3, 2), W.uniform_edges(0, 10e3, 2),
                      W.uniform_edges(0, H, nelz), (True, True))
    ctx = nhsem.Context(mesh, W.Physics(sponge_z0=0.75 * H, sponge_tau=0.01))
    z = ctx.nh_lattice_coords()[2]
    ctx.nh_set_reference(*W.constant_n_reference(z))
    rng = np.random.default_rng(5 * N + nelz)
    b = rng.standard_normal((5, ctx.nz, ctx.nx * ctx.ny)) * np.array([1e-3, 1, 1, 0.1, 0.3])[:, None, None]
    ncol, mr = ctx.nx * ctx.ny, 3
    it = torch.zeros(ncol, dtype=torch.int32, device="cuda")

    def solve(v):
        x, st = ctx.nh_column_solve(0.4, torch.from_numpy(v.reshape(5, -1)).cuda(), restart=restart, max_restarts=mr,
                                    rtol=1e-3, iters=it, schur=schur, check=False)
        return x.cpu().numpy().reshape(b.shape), st, it.cpu().numpy().copy()

    x, st, n = solve(b)
    assert st.not_converged == 0
    rest = np.arange(ncol) != 2
    for bad in (np.inf, -np.inf, np.nan):
        c = b.copy()
        c[field, level, 2] = bad
        y, st, m = solve(c)
        assert st.not_converged == 1 and m[2] < 0, (bad, m[2])
        assert not np.all(np.isfinite(y[:, :, 2]))
        np.testing.assert_array_equal(m[rest], n[rest])
        np.testing.assert_array_equal(y[:, :, rest], x[:, :, rest])


# a reduced system with a NaN takes one step a cycle in every column of the wavefront,
# so that such a column costs the solve no more than the others do
@pytest.mark.parametrize("N,nelz", [(2, 1), (3, 5), (4, 16), (5, 10), (6, 2), (6, 10), (4, 17)])
@pytest.mark.parametrize("restart,mr", [(10, 0), (10, 7)])
def test_nan_ends_a_cycle(N, nelz, restart, mr):
    import torch
    from paper_2504_08157_amd import nhsem
    mesh = W.MeshSpec((2, 1, nelz), N, W.uniform_edges(0, 20e3, 2), W.uniform_edges(0, 10e3, 1),
                      W.uniform_edges(0, 15e3, nelz), (True, True))
    ctx = nhsem.Context(mesh, W.Physics())
    ctx.nh_set_reference(*W.constant_n_reference(ctx.nh_lattice_coords()[2]))
    ncol = ctx.nx * ctx.ny
    b = np.full((5, ctx.nz, ncol), 1e-2)
    b[3, 1] = np.nan
    it = torch.zeros(ncol, dtype=torch.int32, device="cuda")
    x, st = ctx.nh_column_solve(0.4, torch.from_numpy(b.reshape(5, -1)).cuda(), restart=restart, max_restarts=mr,
                                iters=it, schur=True, check=False)
    assert st.not_converged == ncol
    np.testing.assert_array_equal(it.cpu().numpy(), -(mr + 1) - 1)
