"""A reservation that does not fit fails with an error, after which the context
holds no pairs (a neighbour list asks for a new evaluation instead of reading
them) and goes on as before."""
import pytest
import torch

import diskgen
from test_gpu_parity import T

pytestmark = pytest.mark.gpu

STATE, HIP = 4, 3  # P3T_ERR_STATE, P3T_ERR_HIP


@pytest.mark.parametrize("n_max", [2048, 100000])  # without and with a larger arena
def test_reserve_that_does_not_fit(gpu, n_max):
    d = diskgen.workload("disk2k_equal")
    ctx = gpu.Context(gpu.Params.defaults())
    pos, vel, mass = T(d.pos), T(d.vel), T(d.mass)
    ro, rs, _ = ctx.compute_cutoffs(pos, vel, mass)
    acc = ctx.evaluate(pos, vel, mass, ro, rs)
    want = ctx.neighbour_list()
    with pytest.raises(gpu.P3TError) as e:
        ctx.reserve(n_max, 1 << 44)  # 128 TiB
    assert e.value.status == HIP
    with pytest.raises(gpu.P3TError) as e:
        ctx.neighbour_list()
    assert e.value.status == STATE
    assert torch.equal(ctx.evaluate(pos, vel, mass, ro, rs), acc)
    for a, b in zip(ctx.neighbour_list(), want):
        assert torch.equal(a, b)
    ctx.reserve(n_max, 1 << 20)
    assert torch.equal(ctx.evaluate(pos, vel, mass, ro, rs), acc)
    ctx.close()
