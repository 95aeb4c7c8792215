"""The isotropic window sweep, forward and transposed, on every tiling it has,
with the kernel that runs asserted: whole-row waves (one and two cells per
lane), segments of 64, 32 and 16 lanes, chunks of whole and of ragged planes,
linear tiles, directions with one cell, a single cell, waves past the grid; and
P0, which no other kernel takes.

Tolerances: at most ten couplings per moment and step, each rounded once, so
2 steps stay below 1e-13 (FP64) and 1e-6 (FP32) of the largest value; BF16
rounds every value twice per step to 2^-9: below 2e-2.  A gradient adds the
products of a few steps: 1e-12 and 1e-4."""
import numpy as np
import pytest

import paper_2004_02833_amd as pm
from oracle import c_oracle

from gpu_util import relerr, say

pytestmark = pytest.mark.gpu

TOL = {pm.PM_FP64: 1e-13, pm.PM_FP32: 1e-6, pm.PM_BF16: 2e-2}
GRAD_TOL = {pm.PM_FP64: 1e-12, pm.PM_FP32: 1e-4}

SHAPES = [(1, 1, 1), (7, 1, 1), (1, 6, 1), (1, 1, 5), (17, 5, 3), (33, 9, 4), (64, 3, 5), (64, 1, 2), (32, 5, 6), (16, 9, 7), (48, 3, 5),
          (96, 2, 3), (128, 3, 5), (128, 1, 2), (160, 2, 5), (160, 3, 3), (67, 64, 1), (100, 5, 3), (130, 3, 2), (65, 3, 7), (500, 2, 3)]


def _problem(N, shape, seed):
    rng = np.random.default_rng(seed)
    sa, ss, q = rng.uniform(0, 2, shape), rng.uniform(0, 2, shape), rng.uniform(0, 1, shape)
    u0 = rng.standard_normal(((N + 1) ** 2,) + shape)
    u0 = (u0.astype(np.float32).view(np.uint32) & 0xffff0000).view(np.float32).astype(np.float64)  # exact in bfloat16
    return sa, ss, q, u0


@pytest.mark.parametrize("N,nx,ny,nz", [(10,) + s for s in SHAPES] + [(0, 5, 4, 3), (0, 64, 2, 3), (13, 20, 9, 5), (13, 128, 3, 2)])
def test_window_forward(N, nx, ny, nz):
    shape = (nz, ny, nx)
    sa, ss, q, u0 = _problem(N, shape, 100 * N + nx + ny)
    h = 1.0 / max(8, max(shape))
    ref = c_oracle.run(N, shape, h, 0.5 * h, sa, ss, q, u0, 2)
    for prec in TOL:
        pm.pm_set_precision(prec)
        pm.pm_init(N, nx, ny, nz, h, 0.5 * h, sa, ss, q)
        try:
            assert pm.pm_sweep_kind() == pm.PM_SWEEP_WINDOW
            for i in range((N + 1) ** 2):
                pm.pm_write(i, u0[i])
            pm.pm_step(2)
            got = np.stack([pm.pm_read(i) for i in range((N + 1) ** 2)])
        finally:
            pm.pm_finalize()
        e = relerr(got, ref)
        say("window P%d %dx%dx%d prec %d: %.2e" % (N, nx, ny, nz, prec, e))
        assert e <= TOL[prec]


@pytest.mark.parametrize("prec", list(GRAD_TOL))
@pytest.mark.parametrize("N,nx,ny,nz,nsteps,ck", [(10, 9, 7, 6, 5, 2), (10, 64, 3, 5, 3, 1), (11, 32, 5, 6, 4, 4), (10, 100, 5, 3, 3, 2),
                                                  (10, 128, 3, 5, 3, 3), (10, 1, 6, 1, 3, 2), (0, 5, 4, 3, 4, 2)])
def test_window_gradient(N, nx, ny, nz, nsteps, ck, prec):
    shape = (nz, ny, nx)
    rng = np.random.default_rng(5 * N + nx)
    h = 1.0 / max(8, max(shape))
    _, _, q, u0 = _problem(N, shape, N + nx)
    # voids, thin and thick cells: c tau on both sides of the series switch
    sa, ss = rng.choice([0.0, 1e-9, 0.5, 30.0], shape), rng.choice([0.0, 1.0, 3.0 / h], shape)
    tgt = rng.standard_normal(shape)
    _, ga, gs = c_oracle.grad(N, shape, h, 0.5 * h, sa, ss, q, u0, nsteps, ck, tgt)
    pm.pm_set_precision(prec)
    pm.pm_init(N, nx, ny, nz, h, 0.5 * h, sa, ss, q)
    try:
        assert pm.pm_sweep_kind(transposed=True) == pm.PM_SWEEP_WINDOW
        for i in range((N + 1) ** 2):
            pm.pm_write(i, u0[i])
        pm.pm_set_checkpoint(ck)
        pm.pm_step(nsteps)
        dsa, dss = pm.pm_grad(pm.pm_read(0) - tgt)
    finally:
        pm.pm_finalize()
    say("window gradient P%d %dx%dx%d prec %d: %s %s" % (N, nx, ny, nz, prec, np.abs(dsa - ga).max(), np.abs(dss - gs).max()))
    for got, ref in ((dsa, ga), (dss, gs)):
        assert np.abs(got - ref).max() <= GRAD_TOL[prec] * np.abs(ref).max()
