"""Few radial bins: the radii against the oracle (1e-12 relative, as the other
cut-off tests), and no slower than with the default 64, whose passes do the same
work per particle and more of it per bin (a tenth allowed for)."""
import time

import numpy as np
import pytest
import torch

import diskgen
from test_gpu_parity import T, gparams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1000, 70000])
@pytest.mark.parametrize("bins", [1, 2, 3, 15, 16, 17])
def test_values(gpu, orc, n, bins):
    d = diskgen.workload("disk256k_masslaw", n)
    p = orc.Params(vran_bins=bins)
    want = orc.cutoffs(d.pos, d.vel, d.mass, p)
    ctx = gpu.Context(gparams(gpu, p))
    got = ctx.compute_cutoffs(T(d.pos), T(d.vel), T(d.mass))
    for g, w in zip(got, want):
        assert np.abs(g.cpu().numpy() / w - 1.0).max() < 1e-12
    ctx.close()


def test_time(gpu):
    d = diskgen.workload("disk256k_masslaw", 1000)
    best = {}
    out = tuple(torch.empty(1000, dtype=torch.float64, device="cuda:0") for _ in range(3))
    args = T(d.pos), T(d.vel), T(d.mass)
    for bins in (64, 1):
        ctx = gpu.Context(gpu.Params.defaults().replace(vran_bins=bins))
        best[bins] = np.inf
        for _ in range(300):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ctx.compute_cutoffs(*args, out=out)
            torch.cuda.synchronize()
            best[bins] = min(best[bins], (time.perf_counter() - t0) * 1e6)
        ctx.close()
    print("us", best)
    assert best[1] < 1.1 * best[64]
