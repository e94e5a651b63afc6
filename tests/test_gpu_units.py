"""Units of length in which a search radius spans thousands of units (km, m):
a disk with its lengths and velocities times 2^20 and G times 2^60 is the same
disk.  Scaling by a power of two commutes with every operation here (monopole
cells, so that no FP32 product leaves the normal range), so the neighbour rows,
labels and clusters are equal, and the accelerations too, times 2^20.  The
entries that pad a list's last tile then lie inside the search radii: they must
not turn up as neighbours.  Eight wavefronts per group, four with whole and
with half wavefront slots, both precisions."""
import numpy as np
import pytest
import torch

import diskgen
from test_gpu_parity import T

pytestmark = pytest.mark.gpu

SCALE = 2.0 ** 20


@pytest.mark.parametrize("n,group,unroll,precision", [(2048, 128, 2, 0), (2048, 128, 8, 1), (8000, 8, 2, 0), (8000, 8, 8, 1),
                                                      (80001, 96, 4, 0), (80001, 96, 2, 1)])
def test_large_units(gpu, n, group, unroll, precision):
    d = diskgen.workload("disk2k_equal" if n < 80000 else "disk256k_masslaw", n)
    out = []
    for s in (1.0, SCALE):
        p = gpu.Params.defaults().replace(G=s ** 3, theta=0.5, multipole=1, precision=precision, n_group_max=group,
                                          n_leaf_max=min(16, group))
        ctx = gpu.Context(p)
        ctx.set_kernel_config(force_unroll=unroll)
        pos, vel, mass = T(d.pos * s), T(d.vel * s), T(d.mass)
        ro, rs, _ = ctx.compute_cutoffs(pos, vel, mass)
        ctx.build_tree(pos, vel, mass, ro, rs)
        acc = ctx.compute_soft_force()
        rp, col, lab = ctx.neighbour_list()
        out.append((acc / s, ro / s, rp, col, lab, *ctx.clusters(lab), rs))
        ctx.close()
    assert float(out[1][-1].min()) > 1000.0  # the padding's distance from a group starts at this
    print("pairs", out[0][3].shape[0])
    for a, b in zip(out[0][:-1], out[1][:-1]):
        assert torch.equal(a, b)
    col = out[1][3].cpu().numpy()
    assert col.shape[0] > 0 and col.min() >= 0 and col.max() < n
