"""The kernel that pm_init chooses for grids on both sides of each line: a grid
must not move to a kernel that is slower for it."""
import numpy as np
import pytest

import paper_2004_02833_amd as pm
from oracle import c_oracle

from gpu_util import relerr, say

pytestmark = pytest.mark.gpu

W, T, L = pm.PM_SWEEP_WINDOW, pm.PM_SWEEP_TILE, pm.PM_SWEEP_LOW


def _kinds(prec, N, nx, ny, nz):
    f = np.full(nx * ny * nz, 0.5)
    pm.pm_set_precision(prec)
    pm.pm_init(N, nx, ny, nz, 0.01, 0.005, f, f)
    try:
        return pm.pm_sweep_kind(), None if prec == pm.PM_BF16 else pm.pm_sweep_kind(transposed=True)
    finally:
        pm.pm_finalize()


@pytest.mark.parametrize("prec,N,nx,ny,nz,kind", [
    # rows of one or two cells: more padding than values in a box
    (pm.PM_FP64, 7, 1, 512, 512, W), (pm.PM_FP64, 8, 1, 1, 400000, W), (pm.PM_FP64, 7, 2, 512, 512, T),
    (pm.PM_FP32, 8, 1, 1, 400000, W), (pm.PM_FP32, 8, 2, 512, 512, W), (pm.PM_FP32, 12, 5, 300, 300, W),
    # FP32 rows of up to 64 cells, few boxes and many
    (pm.PM_FP32, 12, 20, 130, 97, W), (pm.PM_FP32, 19, 33, 90, 61, W), (pm.PM_FP32, 12, 48, 80, 80, T),
    (pm.PM_FP32, 9, 16, 201, 160, T), (pm.PM_FP32, 8, 40, 200, 200, T), (pm.PM_FP32, 25, 33, 130, 111, T),
    # FP32 planes on cache lines, boxes with idle lanes
    (pm.PM_FP32, 9, 96, 96, 96, W), (pm.PM_FP32, 14, 96, 96, 96, T), (pm.PM_FP32, 9, 128, 64, 64, T),
    (pm.PM_FP32, 9, 250, 61, 36, T), (pm.PM_FP32, 12, 512, 512, 1, T),
    # low orders, small grids
    (pm.PM_FP64, 4, 64, 64, 64, L), (pm.PM_FP32, 7, 64, 64, 64, L), (pm.PM_BF16, 6, 64, 64, 64, L), (pm.PM_BF16, 10, 64, 64, 64, W),
    (pm.PM_FP64, 12, 30, 30, 30, W), (pm.PM_FP64, 12, 64, 64, 64, T), (pm.PM_FP64, 19, 701, 20, 20, T),
    # P0 has no dual moments
    (pm.PM_FP64, 0, 64, 64, 64, W), (pm.PM_FP32, 0, 128, 128, 128, W),
    # FP64 passes that just overflow the chip
    (pm.PM_FP64, 19, 30, 70, 70, W), (pm.PM_FP64, 19, 50, 50, 50, T), (pm.PM_FP64, 19, 56, 56, 56, T), (pm.PM_FP64, 21, 30, 70, 70, T)])
def test_forward_kernel(prec, N, nx, ny, nz, kind):
    assert _kinds(prec, N, nx, ny, nz)[0] == kind


@pytest.mark.parametrize("prec,N,nx,ny,nz,kind", [
    (pm.PM_FP64, 4, 64, 64, 64, L), (pm.PM_FP64, 5, 64, 64, 64, T), (pm.PM_FP64, 5, 161, 45, 33, T), (pm.PM_FP64, 5, 56, 56, 56, W),
    (pm.PM_FP64, 6, 48, 48, 48, W), (pm.PM_FP64, 5, 1, 512, 512, W), (pm.PM_FP64, 7, 64, 64, 64, T), (pm.PM_FP64, 7, 30, 30, 30, W),
    (pm.PM_FP32, 4, 64, 64, 64, L), (pm.PM_FP32, 5, 64, 64, 64, T), (pm.PM_FP32, 7, 128, 64, 64, T), (pm.PM_FP32, 6, 60, 60, 60, T),
    (pm.PM_FP32, 7, 20, 130, 97, W), (pm.PM_FP32, 7, 33, 130, 111, W), (pm.PM_FP32, 5, 32, 32, 32, W), (pm.PM_FP32, 5, 5, 200, 200, W)])
def test_transposed_kernel(prec, N, nx, ny, nz, kind):
    assert _kinds(prec, N, nx, ny, nz)[1] == kind


@pytest.mark.parametrize("prec,N,nx,ny,nz,nsteps,ck", [
    (pm.PM_FP64, 5, 161, 45, 33, 5, 2), (pm.PM_FP64, 6, 64, 62, 66, 3, 3), (pm.PM_FP32, 5, 130, 60, 60, 3, 1), (pm.PM_FP32, 6, 61, 60, 60, 5, 2),
    (pm.PM_FP32, 7, 128, 64, 63, 1, 3)])
def test_gradient_of_low_order_contexts_on_the_tile_sweep(prec, N, nx, ny, nz, nsteps, ck):
    """Low-order forward sweeps under tile transposes, against the oracle: the
    sums of a few steps stay below 1e-12 (FP64) and 1e-4 (FP32)."""
    shape = (nz, ny, nx)
    rng = np.random.default_rng(11 * N + nx)
    h = 1.0 / max(shape)
    # voids, thin and thick cells: c tau on both sides of the series switch
    sa, ss = rng.choice([0.0, 1e-9, 0.5, 30.0], shape), rng.choice([0.0, 1.0, 3.0 / h], shape)
    q, tgt = rng.uniform(0, 1, shape), rng.standard_normal(shape)
    u0 = rng.standard_normal(((N + 1) ** 2,) + shape).astype(np.float32).astype(np.float64)
    _, ga, gs = c_oracle.grad(N, shape, h, 0.5 * h, sa, ss, q, u0, nsteps, ck, tgt)
    pm.pm_set_precision(prec)
    pm.pm_init(N, nx, ny, nz, h, 0.5 * h, sa, ss, q)
    try:
        assert (pm.pm_sweep_kind(), pm.pm_sweep_kind(transposed=True)) == (L, T)
        for i in range((N + 1) ** 2):
            pm.pm_write(i, u0[i])
        pm.pm_set_checkpoint(ck)
        pm.pm_step(nsteps)
        dsa, dss = pm.pm_grad(pm.pm_read(0) - tgt)
    finally:
        pm.pm_finalize()
    e = relerr(dsa, ga), relerr(dss, gs)
    say("tile gradient of low order P%d %dx%dx%d prec %d: %.2e %.2e" % ((N, nx, ny, nz, prec) + e))
    assert max(e) <= (1e-12 if prec == pm.PM_FP64 else 1e-4)
