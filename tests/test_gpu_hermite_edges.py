"""Clusters of one workgroup (65 to 1024 members) and of one wavefront at the
sizes where the members per thread, the lanes per member, the last wavefront and the number of due members per step
change, against the oracle: equal block-step counts, states to the 1e-12 of
the percolated path's test (both sides add the same terms, at most 1024 of
them in another order; the oracle's own states move by 1.3e-15 when its input moves by
1e-15).  The disk's members are due together; a pair and a triple put inside
the changeover region of each cluster add steps with two to five members due.
The state does not depend on whether energies are asked for."""
import numpy as np
import pytest
import torch

import diskgen
from test_gpu_parity import T, gparams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(65, 1, 127, 128, 2, 129), (191, 192, 193, 3, 255, 256), (257, 16, 512, 66),
                                   (513, 64, 1024), (3, 4, 5, 6, 7, 8, 9, 10), (8, 15, 16, 5, 17, 32, 33)])
def test_cluster_sizes(gpu, orc, sizes):
    d = diskgen.workload("disk2k_equal")
    p = orc.Params(eta=0.02, eta0=0.002)
    ro, _, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ptr = np.r_[0, np.cumsum(sizes)].astype(np.int32)
    members = np.random.default_rng(sum(sizes)).permutation(d.n)[: ptr[-1]].astype(np.int32)
    x0, v0 = d.pos.copy(), d.vel.copy()
    for a, b in zip(ptr[:-1], ptr[1:]):
        k = b - a
        groups = ((0, 1), (k // 2, k - 2, k - 1)) if k >= 64 else ((0, 1),) if k > 1 else ()
        for f, g in zip((0.2, 0.4), groups):
            lead = members[a + g[0]]
            for axis, o in enumerate(g[1:]):
                i = members[a + o]
                x0[:, i], v0[:, i] = x0[:, lead], v0[:, lead]
                x0[axis, i] += f * ro[lead]
    xo, vo, e0, e1, ns, st = orc.hermite_clusters(x0, v0, d.mass, ro, ptr, members, p)
    assert st == 0
    ctx = gpu.Context(gparams(gpu, p))
    out = []
    for energy in (True, False):
        pos, vel = T(x0), T(v0)
        err, nst = ctx.hermite_cluster_step(pos, vel, T(d.mass), T(ro), T(ptr, torch.int32), T(members, torch.int32),
                                            steps=True, energy=energy)
        out.append((pos, vel))
        assert np.array_equal(nst.cpu().numpy(), ns)
        if energy:
            eo = np.abs(e1 - e0) / np.abs(e0)
            assert np.all(np.abs(err.cpu().numpy() - eo) <= np.maximum(0.05 * eo, 1e-13))
    print("steps", ns, "max|dx|", np.abs(out[0][0].cpu().numpy() - xo).max())
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert np.abs(out[0][0].cpu().numpy() - xo).max() < 1e-12 and np.abs(out[0][1].cpu().numpy() - vo).max() < 1e-12
    ctx.close()
