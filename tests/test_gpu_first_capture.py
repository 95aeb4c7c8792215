"""A process whose first sweep is queued under HIP graph capture: the context
has loaded the sweep kernels' code, so the capture holds, and its replays
equal eager steps bit for bit (low-order sweep, tile sweep)."""
import os
import subprocess
import sys

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

CODE = """
import sys, numpy as np, torch
torch.zeros(1, device="cuda")
import paper_2004_02833_amd as pm
N, nx, ny, nz, prec = map(int, sys.argv[1:])
shape, V, reps = (nz, ny, nx), (N + 1) ** 2, 3
rng = np.random.default_rng(N)
sa, ss, q = rng.uniform(0, 0.5, shape), rng.uniform(0, 1, shape), rng.uniform(0, 1, shape)
u = rng.normal(size=(V,) + shape)
stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()

def begin():
    pm.pm_set_precision(prec)
    pm.pm_init(N, nx, ny, nz, 1 / 64, 0.5 / 64, sa, ss, q)
    for i in range(V):
        pm.pm_write(i, u[i])

def state():
    return np.stack([pm.pm_read(i) for i in range(V)])

begin()
pm.pm_bind_stream(stream.cuda_stream)
torch.cuda.synchronize()
with torch.cuda.graph(graph, stream=stream):
    pm.pm_step(1)
got = []
for _ in range(reps):
    graph.replay()
    torch.cuda.synchronize()
    pm.pm_total()
    got.append(state())
pm.pm_bind_stream(None)
pm.pm_finalize()
begin()
for k in range(reps):
    pm.pm_step(1)
    assert np.array_equal(got[k], state()), k
pm.pm_finalize()
print("replays equal")
"""


@pytest.mark.parametrize("N,nx,ny,nz,prec", [(3, 16, 12, 10, 0), (9, 80, 41, 27, 0), (4, 64, 92, 92, 1)])
def test_first_sweep_under_capture(N, nx, ny, nz, prec):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, PYTHONPATH=root)
    say("first sweep under capture: P%d %dx%dx%d prec %d" % (N, nx, ny, nz, prec))
    p = subprocess.run([sys.executable, "-c", CODE] + [str(v) for v in (N, nx, ny, nz, prec)],
                       capture_output=True, text=True, env=env, timeout=100)
    assert p.returncode == 0, p.stderr[-2000:]
    assert "replays equal" in p.stdout
