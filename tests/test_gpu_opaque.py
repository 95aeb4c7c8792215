"""Gradients of a medium with opaque cells: sigma_a at the largest double, so
that the mean of two such cells overflows and beta is exactly 0.  Such a point
passes nothing on, as a point of sigma_a = 1e200 does (beta 1e-200 against
values of order 1), so both media must give the same gradient to the last
rounding, in every form of the transposed sweep."""
import numpy as np
import pytest

import paper_2004_02833_amd as pm

from gpu_util import say

pytestmark = pytest.mark.gpu


def _grad(N, shape, prec, g, opaque):
    nz, ny, nx = shape
    rng = np.random.default_rng(N)
    h = 1.0 / max(shape)
    sa, ss = rng.uniform(0, 1, shape), rng.uniform(0, 1, shape)
    u0 = rng.standard_normal((4,) + shape).astype(np.float32).astype(np.float64)
    sa[1:3, 1:3, 1:4] = opaque
    pm.pm_set_precision(prec)
    pm.pm_set_scattering(g)
    try:
        pm.pm_init(N, nx, ny, nz, h, 0.5 * h, sa, ss)
        for i in range(min(4, (N + 1) ** 2)):
            pm.pm_write(i, u0[i])
        pm.pm_set_checkpoint(2)
        pm.pm_step(5)
        return pm.pm_grad(pm.pm_read(0))
    finally:
        pm.pm_set_scattering(None)
        pm.pm_finalize()


@pytest.mark.parametrize("N,shape,prec,g", [
    (0, (4, 5, 6), pm.PM_FP64, None), (3, (6, 7, 9), pm.PM_FP64, None), (3, (6, 7, 9), pm.PM_FP32, None),
    (3, (6, 7, 9), pm.PM_FP64, [0.5, 0.2]), (11, (5, 6, 7), pm.PM_FP64, None), (11, (5, 6, 7), pm.PM_FP32, None),
    (7, (64, 64, 64), pm.PM_FP64, None), (12, (64, 64, 64), pm.PM_FP32, None)])
def test_gradient_of_opaque_cells(N, shape, prec, g):
    ref = _grad(N, shape, prec, g, 1e200)
    got = _grad(N, shape, prec, g, np.finfo(np.float64).max)
    for a, b in zip(got, ref):
        assert np.isfinite(a).all()
        say("opaque P%d %s prec %d: %.2e" % (N, shape, prec, np.abs(a - b).max()))
        assert np.abs(a - b).max() <= 1e-15 * np.abs(b).max()
