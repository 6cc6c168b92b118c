"""GPU: heat conduction over more geometries than the smaller and than the
larger block table of an iteration launch holds (64, 512), against the same
geometries solved one by one (a geometry's blocks, sums and stop test do not
depend on the batch: they agree to rounding)."""
import numpy as np
import pytest

from inputs import gen
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu
NM = 1e-9


@pytest.mark.parametrize("n", [64, 65, 127, 128, 129, 512, 513])
def test_batch_is_each_alone(n):
    P = require_gpu()
    solvers = []
    for k in range(n):
        # 1 block, or 2 to 9 of 256 cells, in turn: the blocks per XCD change from geometry to geometry
        nx, ny = 4 + k % 5 + 40 * (k % 7 == 3), 5 + k % 3 + 40 * (k % 11 == 2)
        s = np.ones((1, ny, nx), np.uint8)
        s[0, 1 + k % 2, 1] = 0
        solvers.append(P.Solver.from_workload(gen.small_2d(nx, ny, solid=s, n_dir=4, n_mfp=1, L=100 * NM)))
    o = P.default_opts(only_fourier=1, waves_per_group=4)
    k, _ = P.solve_batch(solvers, o)
    pick = sorted({0, 1, 3, 62, 63, min(64, n - 1), n // 2, n - 3, n - 2, n - 1})
    alone = [solvers[i].solve(o)["kappa_fourier"] for i in pick]
    assert np.all(np.isfinite(k)) and np.allclose(np.array(k)[pick], alone, rtol=1e-13, atol=0.0)
