"""pm_write_dev and pm_read_dev against their host forms bit for bit: planes
of whole workgroups and ragged ones, device pointers on 16 bytes and 8 bytes
past it, every storage form."""
import numpy as np
import pytest

import paper_2004_02833_amd as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [pm.PM_FP64, pm.PM_FP32, pm.PM_BF16])
@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 1), (1023, 1, 1), (32, 32, 1), (41, 25, 5), (64, 64, 2)])
def test_device_planes_equal_host_planes(nx, ny, nz, prec):
    import torch
    n = nx * ny * nz
    rng = np.random.default_rng(n)
    x = rng.standard_normal(n)
    x[:: max(1, n // 7)] = 1e-41
    one = np.ones(n)
    pm.pm_set_precision(prec)
    pm.pm_init(2, nx, ny, nz, 0.1, 0.05, one, one)
    try:
        pm.pm_write(1, x)
        host = pm.pm_read(1).reshape(-1)
        for off in (0, 1):
            src = torch.zeros(n + 2, dtype=torch.float64, device="cuda")
            src[off:off + n] = torch.from_numpy(x)
            dst = torch.full((n + 3,), 7.0, dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            pm.pm_write_dev(2, src.data_ptr() + 8 * off)
            pm.pm_read_dev(2, dst.data_ptr() + 8 * off)
            pm.pm_sync()
            got = dst.cpu().numpy()
            assert np.array_equal(got[off:off + n], host)
            assert np.all(got[:off] == 7.0) and np.all(got[off + n:] == 7.0)
            assert np.array_equal(pm.pm_read(2).reshape(-1), host)
    finally:
        pm.pm_finalize()
