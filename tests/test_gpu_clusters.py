"""Cluster CSR and bucket lists at the sizes where their passes change: scan
chunks of 1024, clusters sorted by their thread (up to 12 members), by a
wavefront (up to 1024) and by a workgroup, the caller's own labels, labels
outside [0, n).  Whole numbers: equal to a stable numpy sort."""
import numpy as np
import pytest
import torch

import diskgen
from test_gpu_parity import T, gparams

pytestmark = pytest.mark.gpu


def reference(label):
    order = np.argsort(label, kind="stable").astype(np.int32)
    lab = label[order]
    ptr = np.flatnonzero(np.r_[True, lab[1:] != lab[:-1]]).astype(np.int32)
    return np.r_[ptr, label.shape[0]].astype(np.int32), order


@pytest.mark.parametrize("n,kinds", [(1, 1), (2, 1), (1023, 40), (1024, 1024), (1025, 3), (5000, 1), (70000, 9),
                                     (70000, 5000), ((1 << 20) + 3, 200000)])
def test_clusters_any_labels(gpu, n, kinds):
    rng = np.random.default_rng(n + kinds)
    values = rng.choice(n, size=min(kinds, n), replace=False)
    label = values[rng.integers(0, len(values), n)].astype(np.int32)
    ctx = gpu.Context(gpu.Params.defaults())
    for _ in range(2):  # the counters are left clear
        ptr, mem = ctx.clusters(torch.as_tensor(label, device="cuda:0"))
        rp, rm = reference(label)
        assert np.array_equal(ptr.cpu().numpy(), rp) and np.array_equal(mem.cpu().numpy(), rm)
    ctx.close()


def test_clusters_labels_out_of_range(gpu):
    """Labels that are no particle index keep the order by their low bits."""
    n = 3000
    rng = np.random.default_rng(5)
    label = rng.integers(0, n, n).astype(np.int32)
    label[rng.integers(0, n, 50)] = n + 5  # low 12 bits: above every valid label
    ctx = gpu.Context(gpu.Params.defaults())
    ptr, mem = ctx.clusters(torch.as_tensor(label, device="cuda:0"))
    rp, rm = reference(label)
    assert np.array_equal(ptr.cpu().numpy(), rp) and np.array_equal(mem.cpu().numpy(), rm)
    label = np.minimum(label, n - 1)
    ptr, mem = ctx.clusters(torch.as_tensor(label, device="cuda:0"))
    rp, rm = reference(label)
    assert np.array_equal(ptr.cpu().numpy(), rp) and np.array_equal(mem.cpu().numpy(), rm)
    ctx.close()


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("n,r_cut0", [(4096, 2.0), (4096, 10.0), (3001, 60.0)])
def test_labels_and_hard_part(gpu, orc, n, r_cut0, split):
    """Labels of a ring whose graph holds singles, clusters of a few and of a
    thousand and more members, from both force forms; the hard part's own
    clusters give the same state as the caller's."""
    d = diskgen.dense_ring(n, seed=11)
    p = orc.Params(r_cut0=r_cut0)
    ro, rs, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ctx = gpu.Context(gparams(gpu, p, eta=0.02, eta0=0.002))
    ctx.set_kernel_config(force_split=split)
    args = T(d.pos), T(d.vel), T(d.mass), T(ro), T(rs)
    ctx.build_tree(*args)
    ctx.compute_soft_force()
    _, _, lab = ctx.neighbour_list(labels=True)
    rp_o, col_o = orc.neighbour_rows(d.pos, d.vel, d.mass, ro, rs, p)
    lab_o, _ = orc.labels(rp_o, col_o)
    assert np.array_equal(lab.cpu().numpy(), lab_o)
    sizes = np.bincount(np.bincount(lab_o)[lab_o])
    print("largest cluster", sizes.size - 1)
    if sizes.size > 1025:  # the percolated path is checked elsewhere: the clusters alone
        ptr, mem = ctx.clusters(lab)
        rp, rm = reference(lab_o)
        assert np.array_equal(ptr.cpu().numpy(), rp) and np.array_equal(mem.cpu().numpy(), rm)
        return
    a, b = (T(d.pos), T(d.vel)), (T(d.pos), T(d.vel))
    nc = ctx.hard_step(a[0], a[1], T(d.mass), T(ro))
    ptr, mem = ctx.clusters(lab)
    assert nc == ptr.shape[0] - 1
    ctx.hermite_cluster_step(b[0], b[1], T(d.mass), T(ro), ptr, mem, energy=False)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    ctx.close()
