"""Times of the force phase by class: each one measured where the class has
work, together the launch they share; nothing is computed differently with the
timing on."""
import pytest
import torch

import diskgen
from test_gpu_parity import T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,precision", [(2048, 0), (65536, 1), (131072, 0)])
def test_force_phase_by_class(gpu, n, precision):
    d = diskgen.workload("disk64k_masslaw", n)
    ctx = gpu.Context(gpu.Params.defaults().replace(precision=precision))
    pos, vel, mass = T(d.pos), T(d.vel), T(d.mass)
    ro, rs, _ = ctx.compute_cutoffs(pos, vel, mass)
    acc = ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
    keys = ("ms_near", "ms_far", "ms_cell", "ms_cand")
    assert all(ctx.stats()[k] == 0.0 for k in keys)
    ctx.set_timing(True)
    for cfg in (dict(), dict(force_persistent=0)):
        ctx.set_kernel_config(**cfg)
        timed = ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
        st = ctx.stats()
        print(n, cfg, {k: st[k] for k in (*keys, "ms_force")})
        assert torch.equal(acc, timed)
        assert all(st[k] > 0.0 for k in keys)
        # the launch and nothing else lies between the events of the phase
        assert 0.5 * st["ms_force"] < sum(st[k] for k in keys) <= 1.001 * st["ms_force"]
    ctx.set_kernel_config(force_split=0)
    ctx.evaluate(pos, vel, mass, ro, rs, graph=False)
    assert all(ctx.stats()[k] == 0.0 for k in keys) and ctx.stats()["ms_force"] > 0.0
    ctx.close()
