"""The global solve around its first and last passes: the residual formed with L in one
pass (every order, one and many tiles, ragged), a start given, absent or in the result's
own array, several restart cycles, with and without the column preconditioner."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [(2, (40, 9, 3)), (3, (23, 11, 2)), (4, (17, 10, 4)), (5, (3, 4, 2)), (6, (11, 3, 2))]


@pytest.mark.parametrize("pc", [False, True], ids=["plain", "column_preconditioned"])
@pytest.mark.parametrize("N,nel", CASES)
def test_global_solve_forms(N, nel, pc):
    import torch
    from paper_2504_08157_amd import nhsem
    mesh = W.MeshSpec(nel, N, W.uniform_edges(0, 5e3 * nel[0], nel[0]), W.uniform_edges(0, 5e3 * nel[1], nel[1]),
                      W.stretched_edges(0, 6e3, nel[2], seed=2), (True, False))
    ctx = nhsem.Context(mesh, W.Physics())
    c = ctx.nh_lattice_coords()
    ref = W.constant_n_reference(c[2])
    ctx.nh_set_reference(*ref)
    b = torch.from_numpy(W.smooth_random_state(*c, *ref, seed=3, walls=(False, True))).cuda()
    b0, alpha, rtol = b.clone(), 3.0, 1e-11

    def check(x, st, start):
        # the stopping test is on the residual as computed: its rounding is below rtol / 100
        r = b - (x - alpha * ctx.nh_l3_apply(x))
        assert r.norm() <= 1.01 * rtol * b.norm(), start
        assert st.not_converged == 0 and torch.equal(b, b0)

    x1, st = ctx.nh_global_solve(alpha, b, restart=6, max_restarts=200, rtol=rtol, precondition=pc)
    check(x1, st, "b")
    x2, st = ctx.nh_global_solve(alpha, b, x0=torch.zeros_like(b), restart=6, max_restarts=200, rtol=rtol,
                                 precondition=pc)
    check(x2, st, "zero")
    x3 = 0.5 * b
    _, st = ctx.nh_global_solve(alpha, b, x0=x3, out=x3, restart=6, max_restarts=200, rtol=rtol, precondition=pc)
    check(x3, st, "in place")
    # a start that meets rtol is returned as it is, without an Arnoldi step
    x4, st = ctx.nh_global_solve(alpha, b, x0=x1, restart=6, rtol=2 * rtol, precondition=pc)
    assert st.iters_total == 0 and torch.equal(x4, x1)
