"""The FP64 force with four wavefronts per group at the group sizes where the
layout of a group's particles in the lanes changes (32, 64, 96) and with lists
that end inside a tile, theta = 0: against the oracle's direct sum on sampled
particles and its neighbour rows bit for bit.  The tolerances are those of the
theta = 0 test with 2,048 particles (rms 1e-13, largest 1e-11) times the growth
of a random sum's rounding to 80,000 terms, sqrt(80000 / 2048) = 6.3, rounded
up to 10."""
import numpy as np
import pytest

import diskgen
from test_gpu_parity import T, errs, gparams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,group,unroll", [(1300, 1, 2), (3001, 3, 1), (8191, 8, 8), (26001, 32, 2), (27003, 33, 4),
                                            (52000, 64, 2), (77777, 97, 2), (78001, 97, 4)])
def test_group_layouts(gpu, orc, n, group, unroll):
    d = diskgen.workload("disk256k_masslaw", n)
    p = orc.Params()
    ro, rs, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ctx = gpu.Context(gparams(gpu, p, theta=0.0, multipole=2, n_group_max=group))
    ctx.set_kernel_config(force_split=1, force_unroll=unroll)
    ctx.build_tree(T(d.pos), T(d.vel), T(d.mass), T(ro), T(rs))
    acc = ctx.compute_soft_force().cpu().numpy()
    st = ctx.stats()
    assert st["n_near"] + st["n_far"] == n * (n - 1)
    idx = diskgen.sample_indices(n, 256, 11)
    e = errs(acc[:, idx], orc.soft_acc(d.pos, d.mass, ro, p, idx=idx))
    print(n, group, "eps", e)
    assert e[0] < 1e-12 and e[2] < 1e-10
    rp, col, _ = ctx.neighbour_list(labels=False)
    rp, col = rp.cpu().numpy(), col.cpu().numpy()
    rp_o, col_o = orc.neighbour_rows(d.pos, d.vel, d.mass, ro, rs, p, idx=idx)
    for k, i in enumerate(idx):
        assert np.array_equal(col[rp[i]:rp[i + 1]], col_o[rp_o[k]:rp_o[k + 1]]), i
    ctx.close()
