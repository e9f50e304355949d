"""Column solves on both sides of every line at which the form of the column GMRES
changes: lattices of up to 1024, up to 2048 and more columns, the element counts on
either side of the limits at each order, restarts below, at and above 10."""
import math

import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W
from test_gpu_column_gmres import _direct, _rhs

pytestmark = pytest.mark.gpu

FULL10 = [(2, 8), (2, 9), (3, 10), (3, 11), (4, 1), (4, 3), (4, 4), (4, 6), (4, 7), (5, 1), (5, 6), (5, 7), (5, 12),
          (5, 13), (6, 1), (6, 10), (6, 11), (6, 14), (6, 15)]
CASES = [(N, e, 10, False) for N, e in FULL10] + [
    (2, 2, 20, False), (2, 3, 20, False), (2, 3, 15, False), (2, 4, 15, False), (3, 1, 20, False), (3, 3, 16, False),
    (4, 2, 20, False), (4, 3, 17, False), (4, 4, 11, False), (5, 1, 20, False), (5, 3, 20, False), (5, 3, 13, False),
    (6, 2, 20, False), (6, 3, 20, False), (6, 4, 13, False), (5, 1, 4, False), (6, 3, 5, False), (6, 4, 5, False),
    (6, 6, 3, False), (6, 7, 3, False), (6, 2, 10, True), (6, 3, 10, True)]


@pytest.mark.parametrize("least", [1, 1025, 2049])
@pytest.mark.parametrize("N,nelz,restart,schur", CASES)
def test_column_forms(oracle_mod, N, nelz, restart, schur, least):
    import torch
    from paper_2504_08157_amd import nhsem
    ney = 1 if least == 1 else 32 // N
    nex = max(1, math.ceil(least / (ney * N) / N))   # (nex N + 1) x (ney N) columns
    H = 20e3
    mesh = W.MeshSpec((nex, ney, nelz), N, W.uniform_edges(0, 40e3, nex), W.uniform_edges(0, 30e3, ney),
                      W.stretched_edges(0, H, nelz, seed=3), (False, True))
    ph = W.Physics(f=5e-5, sponge_z0=0.75 * H, sponge_tau=0.01)
    ctx = nhsem.Context(mesh, ph)
    z = ctx.nh_lattice_coords()[2]
    ctx.nh_set_reference(*W.constant_n_reference(z))
    # the column operator does not depend on the horizontal mesh
    one = W.MeshSpec((1, 1, nelz), N, W.uniform_edges(0, 40e3, 1), W.uniform_edges(0, 30e3, 1),
                     W.stretched_edges(0, H, nelz, seed=3), (False, True))
    orc = oracle_mod.Oracle(one, ph)
    orc.set_reference(*W.constant_n_reference(orc.lattice_coords()[2]))
    ncol = ctx.nx * ctx.ny
    assert ncol >= least and (least != 1 or ncol <= 64) and (least != 1025 or ncol <= 1536)
    b = _rhs(ctx, z, 10 * N + nelz)
    bd = torch.from_numpy(b).cuda()
    alpha, rtol = 0.3, 1e-10
    A, B, X = _direct(oracle_mod, orc, alpha, b)
    it = torch.zeros(ncol, dtype=torch.int32, device="cuda")
    x, st = ctx.nh_column_solve(alpha, bd, restart=restart, max_restarts=800, rtol=rtol, iters=it, schur=schur)
    assert st.not_converged == 0 and st.iters_total == int(it.sum())
    x = x.cpu().numpy()
    Xg = np.concatenate([x[f].reshape(orc.nz, -1) for f in (0, 3, 4)])
    # the solver's own test with the oracle's operator (rounding of A x in another order:
    # 1e-13 of ||A|| ||x||, taken column by column)
    res = np.linalg.norm(B - A @ Xg, axis=0)
    bound = rtol * np.linalg.norm(B, axis=0) + 1e-13 * np.linalg.norm(A, 2) * np.linalg.norm(Xg, axis=0)
    assert np.all(res <= bound), (res / bound).max()
    np.testing.assert_array_equal(x[1], b[1])
    np.testing.assert_array_equal(x[2], b[2])
