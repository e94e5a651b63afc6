"""Calls that only launch kernels, recorded by the caller into a graph of their
own as the context's first calls on that stream."""
import pytest
import torch

import diskgen
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1000, 5000])  # within and beyond the arena of a new context
def test_kick_and_radii_in_a_callers_graph(gpu, n):
    d = diskgen.workload("disk2k_equal", n)
    pos, vel, mass = T(d.pos), T(d.vel), T(d.mass)
    acc = torch.randn(3, n, dtype=torch.float64, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(n))
    ctx = gpu.Context(gpu.Params.defaults())
    ctx.reserve(n)
    v = vel.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.kick(acc, v, 0.25)
        out = ctx.compute_cutoffs(pos, v, mass)
    want = vel.clone()
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        ctx.kick(acc, want, 0.25)
        ref = ctx.compute_cutoffs(pos, want, mass)
        torch.cuda.synchronize()
        assert torch.equal(v, want)
        for a, b in zip(out, ref):
            assert torch.equal(a, b)
    ctx.close()
