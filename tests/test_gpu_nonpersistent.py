"""One workgroup per group instead of a queue (force_persistent = 0): the same
bits, also where a workgroup takes several groups (many more groups than
n / (2/3 n_group_max)), and a replayed
evaluation, whose host bound on the groups is n, spends no time on idle
workgroups."""
import time

import numpy as np
import pytest
import torch

import diskgen
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


def evaluate(gpu, args, persistent, **kw):
    ctx = gpu.Context(gpu.Params.defaults().replace(**kw))
    ctx.set_kernel_config(force_persistent=persistent)
    pos, vel, mass, ro, rs = args
    eager = ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
    acc = torch.empty_like(eager)
    best = np.inf
    for _ in range(8):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        ctx.evaluate(pos, vel, mass, ro, rs, out=acc, graph=True)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
        assert torch.equal(acc, eager)
    rp, col, lab = ctx.neighbour_list()
    groups = ctx.stats()["n_groups"]
    ctx.close()
    return (eager, rp, col, lab), groups, best


def peeling_clumps():
    """512 clumps in the cells of a grid that the tree's key bits share: 128
    particles in a cell's corner and ten at 3/4, 3/8, ... of its width, which
    the splits peel off one by one: eleven groups of 138 particles."""
    rng = np.random.default_rng(3)
    cell = np.stack(np.meshgrid(np.arange(32.0), np.arange(16.0), indexing="ij")).reshape(2, -1)
    pos = 1e-5 * rng.random((3, 512, 138))
    pos[:2] += cell[:, :, None]
    pos[0, :, 128:] += 0.75 * 0.5 ** np.arange(10)
    pos = pos.reshape(3, -1)
    pos[:, 0], pos[:, -1] = 0.0, (32.0 * 65535 / 65536, 15.0, 0.0)  # the box is the grid
    return pos


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,group", [(3000, 128), (3000, 1), (90000, 128), (20000, 4), (0, 128)])
def test_same_bits(gpu, n, group, precision):
    if n:
        d = diskgen.workload("disk256k_masslaw", n)
        ctx = gpu.Context(gpu.Params.defaults())
        args = T(d.pos), T(d.vel), T(d.mass)
        args = (*args, *ctx.compute_cutoffs(*args)[:2])
        ctx.close()
    else:
        pos = peeling_clumps()
        n = pos.shape[1]
        one = np.ones(n)
        args = T(pos), T(0.0 * pos), T(1e-9 * one), T(1e-6 * one), T(2e-6 * one)
    kw = dict(precision=precision, n_group_max=group, n_leaf_max=min(16, group))
    (a, ga, _), (b, gb, _) = (evaluate(gpu, args, p, **kw) for p in (1, 0))
    most = 4 * (n // max(1, 2 * group // 3)) + 1024
    print("groups", ga, "workgroups at most", most)
    assert ga == gb and (ga > most) == (n == 512 * 138)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def test_replayed_time(gpu):
    """Half as long again as with the queue is allowed for; a workgroup per
    particle took twice as long."""
    n = 1 << 19
    d = diskgen.workload("disk1m_masslaw", n)
    ctx = gpu.Context(gpu.Params.defaults())
    ro, rs, _ = ctx.compute_cutoffs(T(d.pos), T(d.vel), T(d.mass))
    args = T(d.pos), T(d.vel), T(d.mass), ro, rs
    (_, _, q), (_, _, w) = (evaluate(gpu, args, p, precision=1) for p in (1, 0))
    print("queue", q, "workgroups", w)
    assert w < 1.5 * q
