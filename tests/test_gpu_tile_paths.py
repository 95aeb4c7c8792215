"""The tile sweep, forward and transposed, at the edges of its boxes, with the
kernel that runs asserted in every case: rows of whole cache lines, rows that
start inside a line or a 16-byte chunk, rows cut into segments (inside a line,
inside a chunk, a short last one, more segments than a block of boxes), boxes
hanging over the grid in y and z, directions with one cell and rows of two,
one and several passes with an empty last source degree.  A later change of a
threshold that takes a case to another kernel fails here.

Tolerances: at most ten couplings per moment and step, each rounded once, so
2 steps stay below 1e-13 (FP64) and 1e-6 (FP32) of the largest value; a
gradient adds the products of a few steps: 1e-12 and 1e-4."""
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2004_02833_amd as pm
from oracle import c_oracle
from test_gpu_first_capture import CODE

from gpu_util import relerr, say

pytestmark = pytest.mark.gpu


def _run(N, shape, prec, seed, u0, steps, sa, ss, q, ck=0, tgt=None):
    nz, ny, nx = shape
    h = 1.0 / max(shape)
    pm.pm_set_precision(prec)
    pm.pm_init(N, nx, ny, nz, h, 0.5 * h, sa, ss, q)
    try:
        assert pm.pm_sweep_kind() == pm.PM_SWEEP_TILE
        for i in range((N + 1) ** 2):
            pm.pm_write(i, u0[i])
        if not ck:
            pm.pm_step(steps)
            return np.stack([pm.pm_read(i) for i in range((N + 1) ** 2)])
        assert pm.pm_sweep_kind(transposed=True) == pm.PM_SWEEP_TILE
        pm.pm_set_checkpoint(ck)
        pm.pm_step(steps)
        return pm.pm_grad(pm.pm_read(0) - tgt)
    finally:
        pm.pm_finalize()


@pytest.mark.parametrize("prec,N,nx,ny,nz", [
    (pm.PM_FP64, 7, 64, 66, 62), (pm.PM_FP64, 7, 63, 65, 70), (pm.PM_FP64, 7, 161, 45, 33), (pm.PM_FP64, 9, 128, 41, 39),
    (pm.PM_FP64, 7, 250, 1201, 1), (pm.PM_FP64, 9, 100, 1, 3000), (pm.PM_FP64, 7, 2, 300, 410), (pm.PM_FP64, 7, 17, 95, 101),
    (pm.PM_FP64, 12, 48, 45, 41), (pm.PM_FP64, 9, 701, 20, 20),
    (pm.PM_FP32, 8, 64, 92, 92), (pm.PM_FP32, 8, 250, 61, 36), (pm.PM_FP32, 9, 130, 3200, 1), (pm.PM_FP32, 9, 16, 201, 160),
    (pm.PM_FP32, 12, 48, 79, 80), (pm.PM_FP32, 11, 77, 52, 61), (pm.PM_FP32, 14, 161, 45, 33), (pm.PM_FP32, 8, 1303, 20, 25)])
def test_tile_forward(prec, N, nx, ny, nz):
    shape = (nz, ny, nx)
    rng = np.random.default_rng(1000 * N + nx)
    h = 1.0 / max(shape)
    sa, ss, q = rng.uniform(0, 2, shape), rng.uniform(0, 2, shape), rng.uniform(0, 1, shape)
    u0 = rng.standard_normal(((N + 1) ** 2,) + shape).astype(np.float32).astype(np.float64)
    ref = c_oracle.run(N, shape, h, 0.5 * h, sa, ss, q, u0, 2)
    e = relerr(_run(N, shape, prec, nx, u0, 2, sa, ss, q), ref)
    say("tile P%d %dx%dx%d prec %d: %.2e" % (N, nx, ny, nz, prec, e))
    assert e <= (1e-13 if prec == pm.PM_FP64 else 1e-6)


@pytest.mark.parametrize("prec,N,nx,ny,nz,nsteps,ck", [
    (pm.PM_FP64, 7, 64, 66, 62, 1, 5),     # whole lines; one step: the opening half step follows the seed
    (pm.PM_FP64, 7, 63, 65, 70, 7, 3),     # rows inside 16-byte chunks, a short last segment of steps
    (pm.PM_FP64, 7, 161, 45, 33, 4, 1),    # cut rows, every odd substep between two segments
    (pm.PM_FP64, 12, 18, 95, 101, 3, 2),
    (pm.PM_FP32, 9, 128, 64, 64, 3, 3),    # whole lines
    (pm.PM_FP32, 8, 250, 61, 36, 5, 2),    # cut rows
    (pm.PM_FP32, 11, 77, 52, 61, 3, 1)])
def test_tile_gradient(prec, N, nx, ny, nz, nsteps, ck):
    shape = (nz, ny, nx)
    rng = np.random.default_rng(17 * N + nx)
    h = 1.0 / max(shape)
    # voids, thin and thick cells: c tau on both sides of the series switch
    sa, ss = rng.choice([0.0, 1e-9, 0.5, 30.0], shape), rng.choice([0.0, 1.0, 3.0 / h], shape)
    q, tgt = rng.uniform(0, 1, shape), rng.standard_normal(shape)
    u0 = rng.standard_normal(((N + 1) ** 2,) + shape).astype(np.float32).astype(np.float64)
    _, ga, gs = c_oracle.grad(N, shape, h, 0.5 * h, sa, ss, q, u0, nsteps, ck, tgt)
    dsa, dss = _run(N, shape, prec, nx, u0, nsteps, sa, ss, q, ck, tgt)
    e = relerr(dsa, ga), relerr(dss, gs)
    say("tile gradient P%d %dx%dx%d prec %d: %.2e %.2e" % ((N, nx, ny, nz, prec) + e))
    assert max(e) <= (1e-12 if prec == pm.PM_FP64 else 1e-4)


@pytest.mark.parametrize("prec,N,nx,ny,nz", [(pm.PM_FP64, 5, 131, 60, 60), (pm.PM_FP32, 8, 250, 61, 36)])
def test_tile_nonfinite_values_stay_local(prec, N, nx, ny, nz):
    """An infinity reaches only the moments and cells coupled to it: empty
    source slots, idle lanes and halo chunks of other rows contribute nothing."""
    shape = (nz, ny, nx)
    u0 = np.zeros(((N + 1) ** 2,) + shape)
    at = 20, 25, nx // 2
    u0[(6,) + at] = np.inf
    one = np.ones(shape)
    got = _run(N, shape, prec, 0, u0, 1, one, one, None)
    bad = ~np.isfinite(got)
    assert bad[(6,) + at]
    assert max(np.abs(w - c).max() for w, c in zip(np.nonzero(bad.any(axis=0)), at)) <= 3


@pytest.mark.parametrize("N,nx,ny,nz,prec", [(8, 64, 92, 92, 1), (7, 161, 45, 33, 0)])
def test_first_tile_sweep_under_capture(N, nx, ny, nz, prec):
    """The tile sweep as a process's first one, queued under HIP graph capture."""
    code = CODE.replace("begin()\npm.pm_bind", "begin()\nassert pm.pm_sweep_kind() == pm.PM_SWEEP_TILE\npm.pm_bind")
    assert code != CODE
    env = dict(os.environ, PYTHONPATH=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    say("first tile sweep under capture: P%d %dx%dx%d prec %d" % (N, nx, ny, nz, prec))
    p = subprocess.run([sys.executable, "-c", code] + [str(v) for v in (N, nx, ny, nz, prec)],
                       capture_output=True, text=True, env=env, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    assert "replays equal" in p.stdout
