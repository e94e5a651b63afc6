"""Tree moments at the sizes where the bottom-up pass changes its path: one
particle, one chunk (2048 particles) and its neighbours, more nodes than a
chunk's LDS records (leaves of one and two particles), leaves wider than the
groups, several chunks with and without top records in LDS; and the force
launch with eight and (the many small groups of the last case) four wavefronts
per group.

The reference below builds the same tree (48-bit Morton keys, split at the
highest differing bit), its moments by direct sums over each node's particles,
and walks it per group with the opening rule of the library, in numpy FP64.
Both then sum the same terms, so the forces differ only by rounding: 1e-12 of
the sum of the terms' magnitudes (a centre of mass is off by 2e-16, a cell at
least 1e-3 away), where a wrong box, mass, centre or moment of any node is off
by 1e-6 and more.  The frozen-list force (the same pass over the kept
topology) is the same bit for bit.
"""
import numpy as np
import pytest
import torch

import diskgen
from test_gpu_parity import T, gparams

pytestmark = pytest.mark.gpu
GAMMA, THETA = 0.1, 0.5


def spread(v):
    out = np.zeros_like(v)
    for b in range(16):
        out |= ((v >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b)
    return out


def reference(pos, m, ro, rs, n_leaf, n_group, theta=THETA):
    """(acc, sum of term magnitudes) over the tree's lists."""
    n = m.shape[0]
    lo, ext = pos.min(1, keepdims=True), (pos.max(1) - pos.min(1)).max()
    u = ((pos - lo) * (65535.0 / ext if ext > 0 else 0.0)).astype(np.uint64)
    key = (spread(u[0]) << np.uint64(2)) | (spread(u[1]) << np.uint64(1)) | spread(u[2])
    order = np.argsort(key, kind="stable")
    key = key[order]
    x, mm, r_out, reach = pos[:, order].T, m[order], ro[order], np.maximum(ro, rs)[order]

    def split(a, b):  # last index of the left child of [a, b]
        if key[a] == key[b]:
            d = int(a ^ b).bit_length() - 1
            return (b >> d << d) - 1
        d = int(key[a] ^ key[b]).bit_length() - 1
        lo_ = int(key[b]) >> d << d
        return int(np.searchsorted(key[a:b + 1], np.uint64(lo_))) + a - 1

    cache = {}

    def node(a, b):
        if (a, b) not in cache:
            p, w = x[a:b + 1], mm[a:b + 1]
            M = w.sum()
            c = (w[:, None] * p).sum(0) / M
            s = p - c
            Q = 3.0 * np.einsum("k,ki,kj->ij", w, s, s) - (w * (s * s).sum(1)).sum() * np.eye(3)
            cache[a, b] = p.min(0), p.max(0), c, M, Q, reach[a:b + 1].max()
        return cache[a, b]

    acc, mag = np.zeros((n, 3)), np.zeros(n)

    def group(a, b):
        glo, ghi, _, _, _, gr = node(a, b)
        xi = x[a:b + 1]
        stack, nears = [(0, n - 1)], []
        while stack:
            ca, cb = stack.pop()
            clo, chi, c, M, Q, cr = node(ca, cb)
            gap = np.maximum(np.maximum(clo - ghi, glo - chi), 0.0)
            cg = np.maximum(np.maximum(glo - c, c - ghi), 0.0)
            sep = (gap * gap).sum() > (max(gr, cr) * (1.0 + 1e-12)) ** 2
            cnt = cb - ca + 1
            if sep and cnt > 1 and (chi - clo).max() ** 2 < theta ** 2 * (cg * cg).sum():
                d = c - xi
                r = np.sqrt((d * d).sum(1))[:, None]
                Qd = d @ Q
                dQd = (d * Qd).sum(1, keepdims=True)
                t = M * d / r ** 3 - Qd / r ** 5 + 2.5 * dQd * d / r ** 7
                acc[a:b + 1] += t
                mag[a:b + 1] += np.sqrt((t * t).sum(1))
            elif cnt <= n_leaf:
                nears.append((ca, cb, sep))
            else:
                k = split(ca, cb)
                stack += [(ca, k), (k + 1, cb)]
        for ca, cb, sep in nears:
            d = x[None, ca:cb + 1] - xi[:, None]
            r2 = (d * d).sum(2)
            r2[r2 == 0.0] = np.inf  # the particle itself
            K = np.ones_like(r2)
            if not sep:
                y = np.sqrt(r2) / np.maximum(r_out[a:b + 1, None], r_out[None, ca:cb + 1])
                t = np.clip((y - GAMMA) / (1.0 - GAMMA), 0.0, 1.0)
                K = t ** 4 * (35.0 + t * (-84.0 + t * (70.0 - 20.0 * t)))
            f = mm[None, ca:cb + 1] * K / r2 ** 1.5
            acc[a:b + 1] += (f[:, :, None] * d).sum(1)
            mag[a:b + 1] += (f * np.sqrt(np.where(np.isinf(r2), 0.0, r2))).sum(1)

    def groups(a, b):
        if b - a + 1 <= n_group:
            group(a, b)
        else:
            k = split(a, b)
            groups(a, k)
            groups(k + 1, b)

    groups(0, n - 1)
    out, om = np.empty((3, n)), np.empty(n)
    out[:, order], om[order] = acc.T, mag
    return out, om


@pytest.mark.parametrize("n,n_leaf,n_group,top_slots", [
    (1, 16, 128, 4096), (2, 1, 1, 4096), (3, 16, 2, 4096), (130, 16, 128, 4096), (2047, 1, 128, 4096),
    (2048, 16, 128, 4096), (2049, 2, 64, 4096), (4099, 200, 64, 4096), (9001, 16, 128, 4096), (9001, 4, 128, 2),
    (6100, 8, 8, 4096),
])
def test_moments_edges(gpu, orc, n, n_leaf, n_group, top_slots):
    d = diskgen.workload("disk2k_equal", n)
    p = orc.Params()
    ro, rs, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ctx = gpu.Context(gparams(gpu, p, theta=THETA, multipole=2, n_leaf_max=n_leaf, n_group_max=n_group))
    ctx.set_kernel_config(top_slots=top_slots)
    ctx.build_tree(T(d.pos), T(d.vel), T(d.mass), T(ro), T(rs))
    acc = ctx.compute_soft_force()
    assert torch.equal(acc, ctx.soft_force_frozen(T(d.pos), T(d.mass)))
    ref, mag = reference(d.pos, d.mass, ro, rs, n_leaf, n_group)
    off = np.sqrt(((acc.cpu().numpy() - ref) ** 2).sum(0))
    print(n, n_leaf, n_group, top_slots, (off / np.maximum(mag, 1e-300)).max())
    assert (off <= 1e-12 * mag).all()
    ctx.close()


@pytest.mark.parametrize("name,n", [("disk64k_masslaw", 65537), ("disk64k_masslaw", 262144),
                                    ("disk64k_masslaw", 262145), ("disk1m_masslaw", (1 << 20) + 5000)])
def test_sort_sizes(gpu, orc, name, n):
    """Around the sizes where the Morton sort changes its tiles and launches:
    a lost or doubled particle changes the forces and neighbour rows of the
    sampled particles, keys out of order make boxes that span the disk and
    lists many times longer (about 800 interactions per particle here).  Force
    bars of a large disk at theta = 0.5: 2e-3 rms, 5e-4 global."""
    d = diskgen.workload(name, n)
    p = orc.Params()
    ro, rs, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ctx = gpu.Context(gparams(gpu, p, theta=THETA, multipole=2))
    ctx.build_tree(T(d.pos), T(d.vel), T(d.mass), T(ro), T(rs))
    acc = ctx.compute_soft_force().cpu().numpy()
    st = ctx.stats()
    assert (st["n_near"] + st["n_far"] + st["n_cell"]) / n < 2000
    idx = diskgen.sample_indices(n, 512, 7)
    ref = orc.soft_acc(d.pos, d.mass, ro, p, idx=idx)
    num, den = ((acc[:, idx] - ref) ** 2).sum(0), (ref ** 2).sum(0)
    assert np.sqrt(np.mean(num / den)) < 2e-3 and np.sqrt(num.sum() / den.sum()) < 5e-4
    ctx.close()


@pytest.mark.parametrize("theta,n_leaf", [(0.0, 16), (0.1, 1)])
def test_walk_lists_beyond_lds(gpu, orc, theta, n_leaf):
    """Lists, stacks and ranges longer than the walk keeps in LDS (theta = 0
    opens every node; leaves of one particle make a range each).  theta = 0 is the direct sum to rounding (1e-13
    rms); at theta = 0.1 the numpy reference's terms, as above."""
    d = diskgen.workload("disk2k_equal", 6000)
    p = orc.Params()
    ro, rs, _ = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ctx = gpu.Context(gparams(gpu, p, theta=theta, multipole=2, n_leaf_max=n_leaf))
    ctx.build_tree(T(d.pos), T(d.vel), T(d.mass), T(ro), T(rs))
    acc = ctx.compute_soft_force().cpu().numpy()
    if theta == 0.0:
        ref = orc.soft_acc(d.pos, d.mass, ro, p)
        e = ((acc - ref) ** 2).sum(0) / (ref ** 2).sum(0)
        assert np.sqrt(e.mean()) < 1e-13 and ctx.stats()["n_near"] + ctx.stats()["n_far"] == d.n * (d.n - 1)
    else:
        ref, mag = reference(d.pos, d.mass, ro, rs, n_leaf, 128, theta)
        assert (np.sqrt(((acc - ref) ** 2).sum(0)) <= 1e-12 * mag).all()
    ctx.close()
