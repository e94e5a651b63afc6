"""Cut-off radii at the sizes and bin counts where the bin pass changes its
split (workgroup ranges, 256 accumulator columns or fewer), individual and
shared: 1e-12 relative to the oracle (the bars of the other radius tests: bin
sums in another order, device log and cbrt within an ulp), and the
allocation-free entry point equal bit for bit."""
import numpy as np
import pytest
import torch

import diskgen
from test_gpu_parity import T, gparams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n,bins", [(1, 64), (5, 1), (1023, 3), (1025, 64), (4097, 65), (5000, 256), (70001, 100),
                                    (300000, 64)])
def test_cutoffs_edges(gpu, orc, n, bins, mode):
    d = diskgen.workload("disk64k_masslaw", n)
    p = orc.Params(vran_bins=bins, cutoff_mode=mode)
    ref = orc.cutoffs(d.pos, d.vel, d.mass, p)
    gp = gparams(gpu, p, cutoff_mode=mode)
    ctx = gpu.Context(gp)
    got = ctx.compute_cutoffs(T(d.pos), T(d.vel), T(d.mass))
    for a, b in zip(got, ref):
        assert (np.abs(a.cpu().numpy() - b) <= 1e-12 * np.abs(b)).all()
    out = tuple(torch.empty_like(got[0]) for _ in range(3))
    gpu.compute_cutoffs_noalloc(gp, T(d.pos), T(d.vel), T(d.mass), out)
    assert all(torch.equal(a, b) for a, b in zip(got, out))
    ctx.close()
