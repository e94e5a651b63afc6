"""A context whose arena was allocated on a busy stream, used on another stream
that does not wait for it: the counters that every pass expects clear are
cleared behind the busy stream's work, and the other stream's calls wait for
that."""
import pytest
import torch

import diskgen
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reserve", [0, 5000])
def test_arena_of_a_busy_stream(gpu, reserve):
    d = diskgen.workload("disk2k_equal", 4096 if reserve else 1000)
    pos, vel, mass = T(d.pos), T(d.vel), T(d.mass)
    ctx = gpu.Context(gpu.Params.defaults())
    ro, rs, _ = ctx.compute_cutoffs(pos, vel, mass)
    acc = ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
    want = (acc, *ctx.neighbour_list(), *ctx.clusters(ctx.neighbour_list()[2]))
    x, v = pos.clone(), vel.clone()
    ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
    nc = ctx.hard_step(x, v, mass, ro)
    ctx.close()
    junk = [torch.full((1 << 22,), 0x01010101, dtype=torch.int32, device="cuda:0") for _ in range(16)]
    torch.cuda.synchronize()
    busy, other = torch.cuda.Stream(), torch.cuda.Stream()
    del junk  # what fresh memory may hold
    torch.cuda.empty_cache()
    with torch.cuda.stream(busy):
        torch.cuda._sleep(200_000_000)  # about a tenth of a second
        ctx = gpu.Context(gpu.Params.defaults())
        if reserve:
            ctx.reserve(reserve)
    with torch.cuda.stream(other):
        acc = ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
        got = (acc, *ctx.neighbour_list(), *ctx.clusters(ctx.neighbour_list()[2]))
        y, u = pos.clone(), vel.clone()
        ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
        assert ctx.hard_step(y, u, mass, ro) == nc
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    assert torch.equal(x, y) and torch.equal(v, u)
    ctx.close()
