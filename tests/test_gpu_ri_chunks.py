"""The RI diagnostic on lattices whose chunks are cut into waves' columns and rows
differently (a row narrower than a wave, exactly one wave, a node more, several
workgroup widths, longer than a chunk; chunks that begin within a row), and the strip
counts at which the final sums are split (a thread per strip, several, less than one)."""
import numpy as np
import pytest

from oracle import ri_velocity as RI
from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu

# (nx, ny) elements, order; lattice rows of 12, 64, 65, 129, 402, 260 and 4104 nodes
CASES = [((6, 5), 2, 1), ((32, 70), 2, 50), ((16, 70), 4, 128), ((32, 41), 4, 255), ((134, 33), 3, 256),
         ((52, 37), 5, 300), ((2052, 3), 2, 700)]


@pytest.mark.parametrize("nel,N,ns", CASES)
def test_ri_chunks(oracle_mod, nel, N, ns):
    import torch
    from paper_2504_08157_amd import nhsem
    per = (nel[0] != 16 and nel[0] != 32 or N == 2, False)
    ext = (1e3 * nel[0], 1e3 * nel[1])
    mesh = W.MeshSpec((nel[0], nel[1], 2), N, W.stretched_edges(0, ext[0], nel[0], seed=2),
                      W.uniform_edges(0, ext[1], nel[1]), W.uniform_edges(0, 6e3, 2), per)
    ctx, orc = nhsem.Context(mesh, W.Physics()), oracle_mod.Oracle(mesh, W.Physics())
    q = np.random.default_rng(ns).normal(size=(5,) + orc.shape)
    rmax = 0.6 * max(ext)
    want = RI.ri_velocity(orc, q, nstrips=ns, rmax=rmax)
    qd = torch.from_numpy(q).cuda()
    cen = ctx.nh_ri_velocity(qd, nstrips=ns, rmax=rmax)["center"].cpu().numpy()
    # sums of up to 3e5 terms of one sign: below 1e-12 of the extent
    assert np.abs(cen - np.stack([want["xc"], want["yc"]])).max() <= 1e-12 * max(ext)
    got = ctx.nh_ri_velocity(qd, nstrips=ns, rmax=rmax,
                             center=torch.from_numpy(np.stack([want["xc"], want["yc"]])).cuda())
    assert got["count"].cpu().numpy().tolist() == want["count"].tolist()
    # means of terms below 6, each to two ulps: 1e-12 is room for the sums' rounding
    assert np.abs(got["ubar"].cpu().numpy() - want["ubar"]).max() <= 1e-12 * np.abs(want["ubar"]).max()
    res = got["result"].cpu().numpy()
    assert abs(res[0] - want["u_ri"]) <= 1e-12 * want["u_ri"] and abs(res[3] - want["umax"]) <= 1e-15 * want["umax"]
    # the height of the same level (the two lattices' own coordinates round differently)
    z = ctx.nh_lattice_coords()[2]
    assert res[1] == want["r_ri"] and res[2] == z[np.argmin(np.abs(z - want["z_ri"]))]
