"""The 3D linear operator where its work is cut differently: lattices narrower than a
64 x 8 tile, exactly one, a node more, and many tiles; chunks of one to many levels
(few tiles take short chunks, many tiles tall ones)."""
import numpy as np
import pytest

from paper_2504_08157_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [((2, 2, 2), 2, (True, True)), ((16, 2, 3), 4, (True, True)), ((16, 2, 3), 4, (False, False)),
         ((43, 11, 5), 3, (True, False)), ((13, 7, 4), 5, (False, True)), ((11, 5, 3), 6, (True, True)),
         ((70, 64, 4), 4, (True, True)), ((47, 90, 5), 4, (False, False))]


@pytest.mark.parametrize("nel,N,per", CASES)
def test_l3_chunks(oracle_mod, nel, N, per):
    import torch
    from paper_2504_08157_amd import nhsem
    ph = W.Physics(sponge_z0=3e3, sponge_tau=0.02)
    mesh = W.MeshSpec(nel, N, W.stretched_edges(0, 5e5, nel[0], seed=1), W.uniform_edges(0, 4e5, nel[1]),
                      W.stretched_edges(0, 6e3, nel[2], seed=2), per)
    ctx, orc = nhsem.Context(mesh, ph), oracle_mod.Oracle(mesh, ph)
    g, o = ctx.nh_lattice_coords(), orc.lattice_coords()
    ctx.nh_set_reference(*W.constant_n_reference(g[2]))
    orc.set_reference(*W.constant_n_reference(o[2]))
    q = W.smooth_random_state(*o, *W.constant_n_reference(o[2]), seed=11, walls=(not per[0], not per[1]))
    got = ctx.nh_l3_apply(torch.from_numpy(q).cuda()).cpu().numpy()
    want = orc.l3_apply(q)
    # 2 (2N + 1)-point stencils and the sums around them: 40 roundings of 1.1e-16,
    # terms up to 50 times their sum
    for f in range(5):
        n = np.linalg.norm(want[f])
        assert np.linalg.norm(got[f] - want[f]) <= 1e-12 * n if n else np.abs(got[f]).max() == 0.0, f
