"""Clusters of many members: the cluster CSR and the hard part's clusters equal
a stable numpy sort whichever way their members are put in order (by thread up
to 12 members, by wavefront up to 320, by a sort of the labels where a
wavefront's clusters are too much work or larger), and the time of a call does
not depend on how many members share a label."""
import time

import numpy as np
import pytest
import torch

import diskgen
from test_gpu_clusters import reference
from test_gpu_parity import T, gparams

pytestmark = pytest.mark.gpu


def labelled(sizes, seed):
    """Labels (a member's index each, as clusters have) of clusters of these sizes."""
    rng = np.random.default_rng(seed)
    n = int(np.sum(sizes))
    which = rng.permutation(np.repeat(np.arange(len(sizes)), sizes))
    first = np.full(len(sizes), n)
    np.minimum.at(first, which, np.arange(n))
    return first[which].astype(np.int32)


@pytest.mark.parametrize("sizes", [[12], [13], [320], [321], [1024], [12] * 64 + [13], [13] * 64, [60] * 9 + [1] * 200,
                                   [320, 1, 1, 40] * 3, [1] * 300 + [320] + [1] * 300 + [321], [13] * 300 + [300], [200] * 64, [2048] * 3 + [1] * 5000,
                                   [70001], [3] * 40000 + [30] * 2])
def test_cluster_sizes(gpu, sizes):
    lab = labelled(sizes, len(sizes))
    rp, rm = reference(lab)
    ctx = gpu.Context(gpu.Params.defaults())
    for _ in range(2):  # nothing is left over for the next call
        ptr, mem = ctx.clusters(torch.as_tensor(lab, device="cuda:0"))
        assert np.array_equal(ptr.cpu().numpy(), rp) and np.array_equal(mem.cpu().numpy(), rm)
    few = labelled([1] * 500 + [2] * 30, 1)
    ptr, mem = ctx.clusters(torch.as_tensor(few, device="cuda:0"))
    rp, rm = reference(few)
    assert np.array_equal(ptr.cpu().numpy(), rp) and np.array_equal(mem.cpu().numpy(), rm)
    ctx.close()


def test_time_does_not_depend_on_the_sizes(gpu):
    """2^20 particles: one class, 9, 512 and 5,000 classes against clusters of
    one to five members.  All take the launches of the counting passes, and at
    most those of a radix sort of 2^20 keys on top, which together are less than
    three times the first alone; five leaves room for the scatter of a shared
    machine."""
    n = 1 << 20
    ctx = gpu.Context(gpu.Params.defaults())

    def us(kinds):
        lab = np.random.default_rng(kinds).integers(0, kinds, n).astype(np.int32)
        lab = torch.as_tensor(lab, device="cuda:0")
        best = np.inf
        for k in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ctx.clusters(lab)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) * 1e6) if k else best
        return best

    base = us(n // 3)
    times = {k: us(k) for k in (1, 9, 512, 5000)}
    print("us", base, times)
    assert all(t < 5.0 * base for t in times.values())
    ctx.close()


@pytest.mark.parametrize("n,r_cut0,cap", [(4096, 10.0, 1024), (4096, 10.0, 300), (1500, 60.0, 1024)])
def test_hard_part_of_a_percolated_ring(gpu, orc, n, r_cut0, cap):
    """A ring whose graph holds clusters of hundreds and more: the hard part's
    own clusters (prepared behind the evaluation, and formed in the call) give
    the state that the caller's sorted clusters give, bit for bit."""
    d = diskgen.dense_ring(n, seed=11)
    p = orc.Params(r_cut0=r_cut0)
    ro, rs, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ctx = gpu.Context(gparams(gpu, p, eta=0.5, eta0=0.05, dt_soft=2.0 ** -10, cluster_cap=cap))
    args = T(d.pos), T(d.vel), T(d.mass), T(ro), T(rs)
    out = []
    for prepared in (True, False):
        ctx.build_tree(*args)
        ctx.compute_soft_force()
        lab = None
        if not prepared:
            lab = ctx.neighbour_list()[2]  # drops what was prepared
        x, v = T(d.pos), T(d.vel)
        ctx.hard_step(x, v, T(d.mass), T(ro))
        out.append((x, v))
    rp, rm = reference(lab.cpu().numpy())
    print("largest cluster", np.diff(rp).max())
    assert np.diff(rp).max() > 320
    x, v = T(d.pos), T(d.vel)
    ctx.hermite_cluster_step(x, v, T(d.mass), T(ro), T(rp, torch.int32), T(rm, torch.int32), energy=False)
    out.append((x, v))
    for a in out[:2]:
        assert torch.equal(a[0], out[2][0]) and torch.equal(a[1], out[2][1])
    ctx.close()
