"""A particle with a cut-off radius of zero (a massless test particle without a
random-velocity term): its pairs have the other particle's cut-off.
The hard part and the kick adjoint against the oracle, with the tolerances of
their other tests (equal block-step counts, states to 1e-12; 1e-12 of the
largest gradient)."""
import numpy as np
import pytest
import torch

import diskgen
from test_gpu_parity import T, gparams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(2, 3, 4, 5, 8), (9, 16, 33, 64), (65, 300), (513, 1024)])
def test_clusters_with_zero_cutoffs(gpu, orc, sizes):
    d = diskgen.workload("disk2k_equal")
    p = orc.Params(eta=0.02, eta0=0.002)
    ro, _, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ptr = np.r_[0, np.cumsum(sizes)].astype(np.int32)
    members = np.random.default_rng(sum(sizes)).permutation(d.n)[: ptr[-1]].astype(np.int32)
    x0, v0 = d.pos.copy(), d.vel.copy()
    for a, b in zip(ptr[:-1], ptr[1:]):
        i, j = members[a], members[a + 1]  # a pair inside the changeover of one of them
        x0[:, j], v0[:, j] = x0[:, i], v0[:, i]
        x0[0, j] += 0.2 * ro[i]
        ro[j] = 0.0
    xo, vo, _, _, ns, st = orc.hermite_clusters(x0, v0, d.mass, ro, ptr, members, p)
    assert st == 0 and np.isfinite(xo).all()
    ctx = gpu.Context(gparams(gpu, p))
    for energy in (True, False):
        pos, vel = T(x0), T(v0)
        _, nst = ctx.hermite_cluster_step(pos, vel, T(d.mass), T(ro), T(ptr, torch.int32), T(members, torch.int32),
                                          steps=True, energy=energy)
        assert np.array_equal(nst.cpu().numpy(), ns)
        assert np.abs(pos.cpu().numpy() - xo).max() < 1e-12 and np.abs(vel.cpu().numpy() - vo).max() < 1e-12
    ctx.close()


@pytest.mark.parametrize("group", [8, 64, 128])
def test_adjoint_with_a_zero_cutoff(gpu, orc, group):
    n = 500
    d = diskgen.workload("disk2k_equal", n)
    p = orc.Params()
    ro, rs, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ro[17] = 0.0
    lam = np.random.default_rng(group).normal(size=(3, n))
    ogx, ogm = orc.soft_adjoint(d.pos, d.mass, ro, lam, p)
    assert np.isfinite(ogx).all() and np.isfinite(ogm).all()
    ctx = gpu.Context(gparams(gpu, p, theta=0.0, multipole=1, n_group_max=group, n_leaf_max=8))
    ctx.build_tree(T(d.pos), T(d.vel), T(d.mass), T(ro), T(rs))
    ctx.compute_soft_force()
    gx, gm = ctx.soft_kick_adjoint(T(lam), 0.5)
    assert np.abs(gx.cpu().numpy() - 0.5 * ogx).max() < 1e-12 * np.abs(0.5 * ogx).max()
    assert np.abs(gm.cpu().numpy() - 0.5 * ogm).max() < 1e-12 * np.abs(0.5 * ogm).max()
    ctx.close()
