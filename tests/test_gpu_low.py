"""The low-order sweep (N <= 9, everything of a cell at once) against the C
oracle: every order it is built for, one and several passes of target degrees,
workgroups of 64 and of 256 lanes, ragged last workgroups, directions with one
cell, targets streamed (state above 128 MB) and not, and its transpose.

Tolerances as for the tile sweep: at most ten couplings per moment and step,
so 2 steps stay below 1e-13 (FP64) and 1e-6 (FP32) of the largest value; BF16
rounds every value twice per step to 2^-9: below 2e-2."""
import numpy as np
import pytest

import paper_2004_02833_amd as pm
from oracle import c_oracle

from gpu_util import gpu_run, relerr, say

pytestmark = pytest.mark.gpu

TOL = {pm.PM_FP64: 1e-13, pm.PM_FP32: 1e-6, pm.PM_BF16: 2e-2}


def _fields(N, shape, seed):
    rng = np.random.default_rng(seed)
    sa, ss, q = rng.uniform(0, 2, shape), rng.uniform(0, 2, shape), rng.uniform(0, 1, shape)
    u0 = rng.standard_normal(((N + 1) ** 2,) + shape)
    u0 = (u0.astype(np.float32).view(np.uint32) & 0xffff0000).view(np.float32).astype(np.float64)  # exact in bfloat16
    return sa, ss, q, u0


@pytest.mark.parametrize("prec", [pm.PM_FP64, pm.PM_FP32, pm.PM_BF16])
@pytest.mark.parametrize("N,nx,ny,nz", [(N, 17, 5, 3) for N in range(1, 10)] + [
    (1, 1, 9, 7), (2, 130, 1, 1), (3, 1, 1, 65), (4, 65, 64, 63), (3, 67, 65, 61), (1, 300, 299, 200), (9, 20, 30, 40)])
def test_low_forward(N, nx, ny, nz, prec):
    shape = (nz, ny, nx)
    sa, ss, q, u0 = _fields(N, shape, 100 * N + nx)
    h = 1.0 / max(shape)
    ref = c_oracle.run(N, shape, h, 0.5 * h, sa, ss, q, u0, 2)
    e = relerr(gpu_run(N, shape, h, 0.5 * h, sa, ss, q, u0, 2, prec=prec), ref)
    say("low P%d %dx%dx%d prec %d: %.2e" % (N, nx, ny, nz, prec, e))
    assert e <= TOL[prec]


@pytest.mark.parametrize("N,nx,ny,nz,nsteps,ck,prec", [
    (1, 9, 8, 7, 5, 2, pm.PM_FP64), (2, 17, 5, 3, 4, 4, pm.PM_FP64), (3, 67, 65, 61, 3, 1, pm.PM_FP64),
    (4, 33, 20, 9, 4, 3, pm.PM_FP64), (4, 33, 20, 9, 4, 3, pm.PM_FP32), (5, 12, 9, 8, 3, 2, pm.PM_FP64),
    (8, 12, 9, 8, 3, 2, pm.PM_FP32)])
def test_low_gradient(N, nx, ny, nz, nsteps, ck, prec):
    shape = (nz, ny, nx)
    _, _, q, u0 = _fields(N, shape, 7 * N + nx)
    rng = np.random.default_rng(N)
    h = 1.0 / max(shape)
    sa = rng.choice([0.0, 1e-9, 0.5, 30.0], shape)
    ss = rng.choice([0.0, 1.0, 3.0 / h], shape)
    tgt = rng.standard_normal(shape)
    L, ga, gs = c_oracle.grad(N, shape, h, 0.5 * h, sa, ss, q, u0, nsteps, ck, tgt)
    pm.pm_set_precision(prec)
    pm.pm_init(N, nx, ny, nz, h, 0.5 * h, sa, ss, q)
    try:
        for i in range((N + 1) ** 2):
            pm.pm_write(i, u0[i])
        pm.pm_set_checkpoint(ck)
        pm.pm_step(nsteps)
        dsa, dss = pm.pm_grad(pm.pm_read(0) - tgt)
    finally:
        pm.pm_finalize()
    e = relerr(dsa, ga), relerr(dss, gs)
    say("low gradient P%d %dx%dx%d prec %d: %.2e %.2e" % ((N, nx, ny, nz, prec) + e))
    assert max(e) <= (1e-12 if prec == pm.PM_FP64 else 1e-4)
