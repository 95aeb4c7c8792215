"""The kernel that pm_init chooses for grids on both sides of each line: a grid
must not move to a kernel that is slower for it."""
import numpy as np
import pytest

import paper_2004_02833_amd as pm

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
    # FP64 passes that just overflow the chip
    (pm.PM_FP64, 19, 30, 70, 70, W), (pm.PM_FP64, 19, 50, 50, 50, T), (pm.PM_FP64, 19, 56, 56, 56, T), (pm.PM_FP64, 21, 30, 70, 70, T)])
def test_forward_kernel(prec, N, nx, ny, nz, kind):
    assert _kinds(prec, N, nx, ny, nz)[0] == kind
