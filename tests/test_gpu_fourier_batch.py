"""GPU: the heat-conduction iterations of a batch against the same geometries
solved one by one: more geometries than one launch takes, 2D and 3D, and sides
from a few cells to more cells than one per thread.

Tolerance: a geometry's blocks, their sums and its stop test do not depend on
the batch, so the two agree to rounding (1e-13)."""
import numpy as np
import pytest

from inputs import gen
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu
NM = 1e-9


def solid2(nx, ny, k):
    s = np.ones((1, ny, nx), np.uint8)
    if k:
        s[0, ny // 3:2 * ny // 3, nx // 4:nx // 2] = 0
    return s


def geometries():
    out = []
    for k in range(66):
        nx, ny = 5 + 3 * k, 70 - k
        out.append(gen.small_2d(nx, ny, solid=solid2(nx, ny, k % 3), n_dir=8, n_mfp=2, L=100 * NM, Ly=100 * NM * ny / nx))
    # 256 x 300: 300 cells a block
    out.append(gen.small_2d(256, 300, solid=solid2(256, 300, 1), n_dir=8, n_mfp=2, L=100 * NM, Ly=100 * NM))
    return out


def geometries_3d():
    out = []
    for k, (nx, ny, nz) in enumerate([(24, 20, 6), (7, 33, 3), (64, 64, 17)]):
        s = np.ones((nz, ny, nx), np.uint8)
        s[:, ny // 3:2 * ny // 3, nx // 3:nx // 2] = k == 1
        out.append(gen.small_3d(nx, ny, nz, solid=s, n_mfp=2))
    return out


@pytest.mark.parametrize("make", [geometries, geometries_3d])
def test_batch_is_each_alone(make):
    P = require_gpu()
    solvers = [P.Solver.from_workload(w) for w in make()]
    o = P.default_opts(only_fourier=1, waves_per_group=4)
    k, _ = P.solve_batch(solvers, o)
    alone = [s.solve(o)["kappa_fourier"] for s in solvers]
    assert np.all(np.isfinite(k)) and np.allclose(k, alone, rtol=1e-13, atol=0.0)
