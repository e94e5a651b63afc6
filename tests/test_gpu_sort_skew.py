"""The sort's time does not depend on how the keys' digits are spread: a disk in
the box of one particle at 1,000 au, whose upper two key digits are then the
same for all others, against the disk alone.  The passes do the same work; a
counter that all keys of a tile share may not make them wait for each other
(half as much again allowed for).  And the sizes at which the passes change:
98,304, 131,072 and 524,288 keys, with values (the tree) and without (clusters of
a caller's classes, against a stable numpy sort)."""
import numpy as np
import pytest
import torch

import diskgen
import test_gpu_tree_edges as tree_edges
from test_gpu_clusters import reference
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65536, 262144])
def test_far_particle(gpu, n):
    d = diskgen.workload("disk256k_masslaw", n)
    ctx = gpu.Context(gpu.Params.defaults())
    ctx.set_timing(True)
    ms = []
    for far in (1.0, 1e3):
        pos, vel = d.pos.copy(), d.vel.copy()
        pos[:, 0], vel[:, 0] = (far, 0.0, 0.0), (0.0, far ** -0.5, 0.0)
        pos, vel, mass = T(pos), T(vel), T(d.mass)
        ro, rs, _ = ctx.compute_cutoffs(pos, vel, mass)
        best = np.inf
        for _ in range(6):
            ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
            best = min(best, ctx.stats()["ms_sort"])
        ms.append(best)
    print(n, "ms", ms)
    assert 0.0 < ms[1] < 1.5 * ms[0]
    ctx.close()


@pytest.mark.parametrize("n", [98304, 98305, 131072, 131073, 524288, 524289])
def test_sizes(gpu, orc, n):
    tree_edges.test_sort_sizes(gpu, orc, "disk1m_masslaw", n)
    lab = np.random.default_rng(n).integers(0, 7, n).astype(np.int32)
    ctx = gpu.Context(gpu.Params.defaults())
    ptr, mem = ctx.clusters(torch.as_tensor(lab, device="cuda:0"))
    rp, rm = reference(lab)
    assert np.array_equal(ptr.cpu().numpy(), rp) and np.array_equal(mem.cpu().numpy(), rm)
    ctx.close()
