"""Column GMRES with z-elements on lanes (columns of at most 16 elements,
restarts up to 20): every order, the element counts at the edges of its lane
layouts, restart lengths of each of its kernels, partly filled column
groups, and the independence of the columns that share a wavefront."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu


def _pair(oracle_mod, N, nelz, per=(False, True), seed=3):
    import torch
    from paper_2504_08157_amd import nhsem
    H = 20e3
    ph = W.Physics(f=5e-5, sponge_z0=0.75 * H, sponge_tau=0.01)
    # N + 1 by N columns: never a multiple of the columns of a wavefront at once
    mesh = W.MeshSpec((1, 1, nelz), N, W.uniform_edges(0, 40e3, 1), W.uniform_edges(0, 30e3, 1),
                      W.stretched_edges(0, H, nelz, seed=seed), per)
    ctx = nhsem.Context(mesh, ph)
    orc = oracle_mod.Oracle(mesh, ph)
    z = ctx.nh_lattice_coords()[2]
    ctx.nh_set_reference(*W.constant_n_reference(z))
    orc.set_reference(*W.constant_n_reference(orc.lattice_coords()[2]))
    ctx.nh_hevi_attach()
    return ctx, orc, z, torch


def _rhs(ctx, z, seed):
    """Right-hand sides that differ from column to column, w = 0 on the walls."""
    rho0, th0 = W.constant_n_reference(z)
    D = np.stack([rho0, np.full_like(rho0, 340.0), th0])
    q = W.random_column_rhs(z, D, ctx.nx * ctx.ny, seed, modes=6).reshape((5,) + ctx.shape)
    q[1] = 1.0 + np.arange(q[1].size).reshape(q[1].shape)
    q[2] = -2.0 - np.arange(q[2].size).reshape(q[2].shape)
    return q


def _direct(oracle_mod, orc, alpha, b):
    nz = orc.nz
    A = np.eye(3 * nz) - alpha * oracle_mod.column_matrix(orc)
    B = np.concatenate([b[f].reshape(nz, -1) for f in (0, 3, 4)])
    return A, B, np.linalg.solve(A, B)


# nelz = 16: the top level in the extra slot; 15: in the last lane (pair); 1:
# one element; restarts 10 (and the Schur form), 7 and 13: a restart shorter
# than the kernel's basis, 20: the longest
SHAPES = [(N, e) for N in (2, 3, 4, 5, 6) for e in (1, 15, 16)] + [(4, 7), (5, 11)]


@pytest.mark.parametrize("restart,schur", [(10, False), (7, False), (13, False), (20, False), (10, True)])
@pytest.mark.parametrize("N,nelz", SHAPES)
def test_lane_gmres_vs_direct(oracle_mod, N, nelz, restart, schur):
    ctx, orc, z, torch = _pair(oracle_mod, N, nelz)
    b = _rhs(ctx, z, 40 + N + nelz)
    bd = torch.from_numpy(b).cuda()
    alpha, rtol = 0.5, 1e-11
    A, B, X = _direct(oracle_mod, orc, alpha, b)
    it = torch.zeros(ctx.nx * ctx.ny, dtype=torch.int32, device="cuda")
    x, st = ctx.nh_column_solve(alpha, bd, restart=restart, max_restarts=400, rtol=rtol, iters=it, schur=schur)
    assert st.not_converged == 0 and st.iters_total == int(it.sum())
    x = x.cpu().numpy()
    Xg = np.concatenate([x[f].reshape(orc.nz, -1) for f in (0, 3, 4)])
    # the solver's own test, with the oracle's operator (rounding of A x in
    # another order: 1e-13 of ||A|| ||x||, taken column by column)
    res = np.linalg.norm(B - A @ Xg, axis=0)
    bound = rtol * np.linalg.norm(B, axis=0) + 1e-13 * np.linalg.norm(A, 2) * np.linalg.norm(Xg, axis=0)
    assert np.all(res <= bound), (res / bound).max()
    np.testing.assert_array_equal(x[1], b[1])
    np.testing.assert_array_equal(x[2], b[2])
    # in place, and from the solution as guess
    y = bd.clone()
    ctx.nh_column_solve(alpha, y, out=y, restart=restart, max_restarts=400, rtol=rtol, schur=schur)
    np.testing.assert_array_equal(y.cpu().numpy(), x)
    x0 = torch.from_numpy(np.ascontiguousarray(np.stack([x[0], x[3], x[4]]))).cuda()
    _, st0 = ctx.nh_column_solve(alpha, bd, x0=x0, restart=restart, rtol=1e-8, schur=schur)
    assert st0.iters_total == 0


@pytest.mark.parametrize("restart,schur", [(10, False), (20, False), (10, True)])
def test_columns_of_a_wave_are_independent(oracle_mod, restart, schur):
    """A zero column, a column of NaN and one that starts from its solution
    leave the other columns' solutions and step counts bitwise unchanged."""
    ctx, orc, z, torch = _pair(oracle_mod, 4, 16)
    b = _rhs(ctx, z, 77)
    ncol = ctx.nx * ctx.ny
    bd = torch.from_numpy(b).cuda()
    it0 = torch.zeros(ncol, dtype=torch.int32, device="cuda")
    it1 = torch.zeros(ncol, dtype=torch.int32, device="cuda")
    x0 = torch.stack([bd[0], bd[3], bd[4]]).contiguous()
    kw = dict(restart=restart, max_restarts=30, rtol=1e-10, schur=schur)
    ref, _ = ctx.nh_column_solve(0.5, bd, x0=x0, iters=it0, **kw)
    mod = bd.clone().view(5, ctx.nz, ncol)
    g = x0.clone().view(3, ctx.nz, ncol)
    sol = ref.view(5, ctx.nz, ncol)
    mod[:, :, 5] = 0.0
    mod[:, :, 10] = float("nan")
    for k, f in enumerate((0, 3, 4)):
        g[k, :, 15] = sol[f, :, 15]
        g[k, :, 5] = 0.0
        g[k, :, 10] = mod[f, :, 10]
    out, st = ctx.nh_column_solve(0.5, mod, x0=g, iters=it1, check=False, **kw)
    got = out.view(5, ctx.nz, ncol)
    keep = [c for c in range(ncol) if c not in (5, 10, 15)]
    assert torch.equal(got[:, :, keep], sol[:, :, keep])
    assert torch.equal(it1[keep], it0[keep]) and st.not_converged == 1
    assert it1[5] == 0 and it1[15] == 0 and it1[10] < 0
    assert torch.count_nonzero(got[:, :, 5]) == 0


@pytest.mark.parametrize("restart", [10, 20])
def test_lane_gmres_wall_values_of_the_guess(oracle_mod, restart):
    """A guess whose wall values of w differ from b's: their rows are the
    identity, and the solve returns b there."""
    ctx, orc, z, torch = _pair(oracle_mod, 3, 16)
    b = _rhs(ctx, z, 5)
    b[3, 0], b[3, -1] = 0.25, -0.5
    bd = torch.from_numpy(b).cuda()
    A, B, X = _direct(oracle_mod, orc, 0.4, b)
    rng = np.random.default_rng(1)
    x0 = torch.from_numpy(X.reshape((3,) + ctx.shape) * (1.0 + 0.1 * rng.normal(size=(3,) + ctx.shape))).cuda()
    x, st = ctx.nh_column_solve(0.4, bd, x0=x0, restart=restart, max_restarts=400, rtol=1e-12)
    Xg = np.concatenate([x.cpu().numpy()[f].reshape(orc.nz, -1) for f in (0, 3, 4)])
    assert np.all(np.linalg.norm(B - A @ Xg, axis=0) <= 2e-12 * np.linalg.norm(B, axis=0)
                  + 1e-13 * np.linalg.norm(A, 2) * np.linalg.norm(Xg, axis=0))


def test_lane_gmres_reports_non_convergence(oracle_mod):
    ctx, orc, z, torch = _pair(oracle_mod, 4, 9)
    bd = torch.from_numpy(_rhs(ctx, z, 6)).cuda()
    it = torch.zeros(ctx.nx * ctx.ny, dtype=torch.int32, device="cuda")
    for restart in (3, 15):
        _, st = ctx.nh_column_solve(3.0, bd, restart=restart, max_restarts=1, rtol=1e-13, iters=it, check=False)
        assert st.not_converged == st.columns and bool((it == -2 * restart - 1).all())
