"""Column GMRES of columns of more than 16 elements: one column per wavefront."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W
from test_gpu_column_gmres import _direct, _pair, _rhs

pytestmark = pytest.mark.gpu


def _check(orc, A, B, b, x, rtol):
    """The solver's own test with the oracle's operator (rounding of A x in another
    order: 1e-13 of ||A|| ||x||, taken column by column); u and v copied."""
    Xg = np.concatenate([x[f].reshape(orc.nz, -1) for f in (0, 3, 4)])
    res = np.linalg.norm(B - A @ Xg, axis=0)
    bound = rtol * np.linalg.norm(B, axis=0) + 1e-13 * np.linalg.norm(A, 2) * np.linalg.norm(Xg, axis=0)
    assert np.all(res <= bound), (res / bound).max()
    np.testing.assert_array_equal(x[1], b[1])
    np.testing.assert_array_equal(x[2], b[2])


# 17 elements, the first column not solved with elements on lanes; 20 and 28: the tallest
# of the register form (3 n_z <= 256) among orders 3 and 4; 25 and 21: the Schur form's
@pytest.mark.parametrize("N,nelz,schur", [(2, 17, False), (4, 17, False), (4, 20, False), (3, 28, False),
                                          (2, 17, True), (4, 17, True), (4, 20, True), (5, 25, True),
                                          (6, 21, True)])
def test_early_stop_takes_no_vector_past_it(oracle_mod, N, nelz, schur):
    """A cycle that stops before its last step leaves the later basis vectors
    unwritten.  The wavefronts before it were of columns of NaN, which their
    registers then hold: the solves converge all the same, and to the same bits
    each time."""
    from paper_2504_08157_amd import nhsem
    ctx, orc, z, torch = _pair(oracle_mod, N, nelz)
    # about 5000 columns of NaN: several waves for every SIMD
    mesh = W.MeshSpec((72 // N, 72 // N, nelz), N, W.uniform_edges(0, 40e3, 72 // N),
                      W.uniform_edges(0, 30e3, 72 // N), W.uniform_edges(0, 20e3, nelz), (False, False))
    wide = nhsem.Context(mesh, W.Physics())
    wide.nh_set_reference(*W.constant_n_reference(wide.nh_lattice_coords()[2]))
    wide.nh_hevi_attach()
    b = _rhs(ctx, z, 60 + N + nelz)
    bd = torch.from_numpy(b).cuda()
    bad = torch.full((5, mesh.U), float("nan"), dtype=torch.float64, device="cuda")
    alpha, rtol = 0.2, 1e-9
    A, B, X = _direct(oracle_mod, orc, alpha, b)
    it = torch.zeros(ctx.nx * ctx.ny, dtype=torch.int32, device="cuda")
    runs = []
    for _ in range(4):
        _, st = wide.nh_column_solve(alpha, bad, restart=10, max_restarts=1, rtol=rtol, schur=schur, check=False)
        assert st.not_converged == st.columns
        x, st = ctx.nh_column_solve(alpha, bd, restart=10, max_restarts=200, rtol=rtol, iters=it, schur=schur,
                                    check=False)
        assert st.not_converged == 0 and int((it % 10 != 0).sum()) > 0
        runs.append((x.cpu().numpy(), it.cpu().numpy()))
    _check(orc, A, B, b, runs[0][0], rtol)
    for x, i in runs[1:]:
        np.testing.assert_array_equal(x, runs[0][0])
        np.testing.assert_array_equal(i, runs[0][1])


# either side of the dispatch: restarts above 20 on short columns, and columns of 17
# elements at every order (3 n_z <= 256: registers; above and at other restarts: LDS)
@pytest.mark.parametrize("N,nelz,restart,schur", [(4, 5, 21, False), (2, 16, 21, False), (4, 16, 40, False),
                                                  (6, 16, 40, False), (2, 17, 10, False), (2, 17, 20, False),
                                                  (2, 17, 10, True), (3, 17, 10, False), (3, 17, 20, False),
                                                  (3, 17, 10, True), (4, 17, 20, False), (5, 17, 10, False),
                                                  (5, 17, 10, True), (6, 17, 20, False), (6, 17, 10, True)])
def test_wave_gmres_vs_direct(oracle_mod, N, nelz, restart, schur):
    ctx, orc, z, torch = _pair(oracle_mod, N, nelz)
    b = _rhs(ctx, z, 20 + N + nelz)
    bd = torch.from_numpy(b).cuda()
    alpha, rtol = 0.5, 1e-11
    A, B, X = _direct(oracle_mod, orc, alpha, b)
    it = torch.zeros(ctx.nx * ctx.ny, dtype=torch.int32, device="cuda")
    x, st = ctx.nh_column_solve(alpha, bd, restart=restart, max_restarts=400, rtol=rtol, iters=it, schur=schur)
    assert st.not_converged == 0 and st.iters_total == int(it.sum())
    x = x.cpu().numpy()
    _check(orc, A, B, b, x, rtol)
    x0 = torch.from_numpy(np.ascontiguousarray(np.stack([x[0], x[3], x[4]]))).cuda()
    _, st0 = ctx.nh_column_solve(alpha, bd, x0=x0, restart=restart, rtol=1e-8, schur=schur)
    assert st0.iters_total == 0


@pytest.mark.parametrize("N,nelz,schur", [(4, 17, False), (4, 17, True), (3, 28, False), (5, 25, True)])
def test_guess_pick_per_column(oracle_mod, N, nelz, schur):
    """The choice of start in columns of more than 16 elements: every other column is
    given its solution (kept: no Arnoldi step), the rest a guess far from it (replaced
    by the default start: its step counts)."""
    ctx, orc, z, torch = _pair(oracle_mod, N, nelz)
    b = _rhs(ctx, z, 80 + N + nelz)
    bd = torch.from_numpy(b).cuda()
    alpha, rtol = 0.3, 1e-9
    A, B, X = _direct(oracle_mod, orc, alpha, b)
    ncol = ctx.nx * ctx.ny
    kw = dict(restart=10, max_restarts=200, rtol=rtol, schur=schur)
    it0 = torch.zeros(ncol, dtype=torch.int32, device="cuda")
    it1 = torch.zeros(ncol, dtype=torch.int32, device="cuda")
    ctx.nh_column_solve(alpha, bd, iters=it0, **kw)
    rng = np.random.default_rng(N)
    g = X.reshape(3, orc.nz, ncol).copy()
    far = 3.0 * g + rng.normal(size=g.shape) * np.abs(g).max(axis=(1, 2), keepdims=True)
    g[:, :, 1::2] = far[:, :, 1::2]
    x, st = ctx.nh_column_solve(alpha, bd, x0=torch.from_numpy(g).cuda(), iters=it1, pick=True, **kw)
    assert st.not_converged == 0
    want = it0.cpu().numpy()
    want[::2] = 0
    np.testing.assert_array_equal(it1.cpu().numpy(), want)
    _check(orc, A, B, b, x.cpu().numpy(), rtol)
