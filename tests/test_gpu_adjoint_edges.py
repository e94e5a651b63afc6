"""The kick adjoint at the group sizes where the places per lane change (32,
64, 96, 128 particles per group) and at list lengths around its tiles of 64
and half tiles of 32, with the tolerances of the adjoint's other tests: 1e-12
against the oracle (FP64, every interaction a pair), 1e-6 against central
differences (cells), 1e-5 mixed against FP64."""
import numpy as np
import pytest

import diskgen
from test_gpu_adjoint import T, fd_check, setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,group", [(2, 1), (33, 16), (65, 31), (96, 32), (97, 33), (500, 64), (1000, 65), (1111, 96),
                                     (2048, 97), (2048, 128)])
def test_group_sizes(gpu, orc, n, group):
    d = diskgen.workload("disk2k_equal", n)
    lam = np.random.default_rng(n + group).normal(size=(3, n))
    ctx, g, acc, ro, p = setup(gpu, orc, d, theta=0.0, multipole=1, n_group_max=group)
    gx, gm = ctx.soft_kick_adjoint(T(lam), 0.5)
    ogx, ogm = orc.soft_adjoint(d.pos, d.mass, ro, lam, p)
    assert np.abs(gx.cpu().numpy() - 0.5 * ogx).max() < 1e-12 * np.abs(0.5 * ogx).max()
    assert np.abs(gm.cpu().numpy() - 0.5 * ogm).max() < 1e-12 * np.abs(0.5 * ogm).max()
    c32 = setup(gpu, orc, d, theta=0.0, multipole=1, n_group_max=group, precision=1)[0]
    hx, hm = c32.soft_kick_adjoint(T(lam), 0.5)
    assert (hx - gx).abs().max() < 1e-5 * gx.abs().max() and (hm - gm).abs().max() < 1e-5 * gm.abs().max()
    if n >= 500:
        ctx, g, _, _, _ = setup(gpu, orc, d, theta=0.5, multipole=1, n_group_max=group)
        gx, gm = ctx.soft_kick_adjoint(T(lam), 1.0)
        assert ctx.stats()["n_cell"] > 0
        wx, wm = fd_check(ctx, g, n, T(lam), diskgen.sample_indices(n, 6, 3), gx, gm, 1e-9)
        assert wx < 1e-6 and wm < 1e-6


def test_nan_cotangent_stays_with_its_pairs(gpu, orc):
    """A NaN cotangent of one particle: that particle's mass gradient has no
    term of its own cotangent (theta = 0), so it stays finite; its partners'
    and its own position gradients are NaN, as the oracle's."""
    n, k = 300, 17
    d = diskgen.workload("disk2k_equal", n)
    lam = np.random.default_rng(1).normal(size=(3, n))
    lam[:, k] = np.nan
    for group in (8, 64, 128):
        ctx, g, acc, ro, p = setup(gpu, orc, d, theta=0.0, multipole=1, n_group_max=group)
        gx, gm = ctx.soft_kick_adjoint(T(lam), 0.5)
        ogx, ogm = orc.soft_adjoint(d.pos, d.mass, ro, lam, p)
        assert np.array_equal(np.isnan(gx.cpu().numpy()), np.isnan(ogx))
        assert np.array_equal(np.isnan(gm.cpu().numpy()), np.isnan(ogm))
        assert np.isfinite(ogm[k])
