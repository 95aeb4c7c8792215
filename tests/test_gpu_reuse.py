"""Contexts that replace each other without pm_finalize take over device
memory and the library's stream: every run equals the same run on a fresh
context bit for bit, across sizes, storage forms, streams and gradients, and
pm_finalize gives the memory back."""
import numpy as np
import pytest

import paper_2004_02833_amd as pm

from gpu_util import say

pytestmark = pytest.mark.gpu

# (N, shape, precision, gradient, own torch stream)
RUNS = [(3, (20, 18, 14), pm.PM_FP64, True, False), (3, (20, 18, 14), pm.PM_FP64, True, True),
        (3, (20, 18, 15), pm.PM_FP64, False, True), (3, (20, 18, 14), pm.PM_FP32, True, False),
        (7, (64, 64, 64), pm.PM_FP64, True, True), (7, (64, 64, 64), pm.PM_FP64, True, False),
        (7, (64, 64, 64), pm.PM_BF16, False, False), (12, (20, 18, 14), pm.PM_FP32, True, True)]


def _run(k, N, shape, prec, grad, own_stream):
    import torch
    rng = np.random.default_rng(k)
    nz, ny, nx = shape
    h = 1.0 / max(shape)
    sa, ss = rng.uniform(0, 1, shape), rng.uniform(0, 1, shape)
    stream = torch.cuda.Stream() if own_stream else None
    pm.pm_bind_stream(stream.cuda_stream if own_stream else None)
    pm.pm_set_precision(prec)
    pm.pm_init(N, nx, ny, nz, h, 0.5 * h, sa, ss, rng.uniform(0, 1, shape))
    for i in range(4):
        pm.pm_write(i, rng.standard_normal(shape))
    if grad:
        pm.pm_set_checkpoint(2)
    pm.pm_step(5)
    out = [pm.pm_read(i) for i in (0, 3, (N + 1) ** 2 - 1)]
    if grad:
        out += list(pm.pm_grad(out[0]))
    return out


def test_replaced_contexts_equal_fresh_ones():
    import torch
    try:
        fresh = []
        for k, r in enumerate(RUNS):
            fresh.append(_run(k, *r))
            pm.pm_bind_stream(None)
            pm.pm_finalize()
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        for k, r in enumerate(RUNS):
            for a, b in zip(_run(k, *r), fresh[k]):
                assert np.array_equal(a, b), r
        pm.pm_bind_stream(None)
        pm.pm_finalize()
        free1 = torch.cuda.mem_get_info()[0]
        say("free before %d after %d" % (free0, free1))
        assert free1 >= free0 - (64 << 20)
    finally:
        pm.pm_bind_stream(None)
        pm.pm_finalize()
