"""The stage launch's column split and tile choice (lattices with few tiles):
bitwise the results of whole columns with another tile (variant 1), at
sizes that take each tile shape with one, several and uneven runs of
elements per column, with walls and without, both precisions."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu

MESHES = [
    (2, 9, 7, 5), (2, 40, 40, 16), (2, 100, 90, 7),
    (3, 10, 10, 8), (3, 33, 27, 7), (3, 61, 45, 14),
    (4, 1, 1, 1), (4, 1, 3, 2), (4, 4, 4, 4), (4, 16, 16, 10), (4, 24, 21, 11), (4, 40, 40, 16), (4, 5, 70, 9),
    (5, 5, 5, 18), (5, 21, 34, 9), (5, 29, 32, 7), (5, 40, 41, 8),
    (6, 10, 10, 6), (6, 15, 4, 7), (6, 24, 23, 5), (6, 40, 40, 4),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("mesh", MESHES, ids=lambda m: "N%d_%dx%dx%d" % m)
def test_split_bitwise_equals_whole_columns(mesh, prec):
    import torch
    from paper_2504_08157_amd import nhsem
    N, nx, ny, nz = mesh
    per = (nx % 2 == 0, ny % 2 == 1)
    m = W.MeshSpec((nx, ny, nz), N, W.uniform_edges(-6e5, 6e5, nx), W.uniform_edges(-6e5, 6e5, ny),
                   W.stretched_edges(0.0, 2e4, nz, seed=4), per)
    ph = W.Physics(f=5e-5, sponge_z0=15e3, sponge_tau=0.02)
    p = nhsem.NH_FP64 if prec == "fp64" else nhsem.NH_FP32_MIXED
    ctx = nhsem.Context(m, ph, precision=p)
    x, y, z = ctx.nh_lattice_coords()
    rho0, th0 = W.constant_n_reference(z)
    ctx.nh_set_reference(rho0, th0)
    rng = np.random.default_rng(sum(mesh))
    heat = torch.from_numpy(1e-3 * rng.normal(size=(2, ctx.U))).cuda()
    ctx.nh_set_forcing(4, [0.0, 10.0], heat)
    # white noise of small amplitude: every node of every field matters
    q = rng.normal(size=(5,) + ctx.shape) * np.array([1e-4, 1.0, 1.0, 0.1, 0.1])[:, None, None, None]
    q[3, 0] = q[3, -1] = 0.0
    q = torch.from_numpy(q).cuda()
    out = []
    for variant in (0, 1):
        ctx.nh_set_tile(variant)
        ctx.nh_set_state(q)
        ctx.nh_rk_step(1.0, 1e-3, 2)
        out.append((ctx.nh_rhs(2.0, q), ctx.nh_get_state()))
    assert bool(torch.isfinite(out[0][1]).all())
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    ctx.close()
