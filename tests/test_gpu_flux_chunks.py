"""GPU: the flux map and the gradient over chunks of systems, at system counts
around the chunks (fewer systems than waves, a part past a multiple of eight)
and cell counts that leave a part of the last block.

Flux: J sums to kappa, kappa_cc = L / (dT V) sum V J_g, both FP64 sums of the
same terms (1e-11).  Gradient: against a central difference of kappa at one
cell (step 1e-4, converged to 1e-12: truncation below 1e-6 of it)."""
import numpy as np
import pytest
import torch

from inputs import gen
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n_dir,n_mfp", [(9, 7, 4, 1), (13, 11, 8, 2), (16, 16, 8, 17), (21, 20, 12, 11)])
def test_flux_and_gradient(nx, ny, n_dir, n_mfp):
    P = require_gpu()
    solid = np.ones((1, ny, nx), np.uint8)
    solid[0, 3:5, 3:6] = 0
    w = gen.small_2d(nx, ny, solid=solid, n_dir=n_dir, n_mfp=n_mfp, Ly=100e-9 * ny / nx)
    s = P.Solver.from_workload(w)
    o = s.opts(precision=0, outer_tol=1e-12, max_outer=4000, inner_tol=1e-13, accel=8, fourier_tol=1e-10)
    r = s.solve(o, want_J=True)
    J = r["J"].cpu().numpy().reshape(ny * nx, -1)
    assert abs(w.L[0] / w.dT * J[:, 0].mean() - r["kappa"]) <= 1e-11 * abs(r["kappa"])
    assert np.all(J[solid.ravel() == 0] == 0.0)
    sig = torch.ones(nx * ny, dtype=torch.float64, device="cuda", requires_grad=True)
    k = P.KappaEff.apply(sig, s, o)
    k.backward()
    g = sig.grad.cpu().numpy()
    assert np.all(g[solid.ravel() == 0] == 0.0)
    c, h = nx + 1, 1e-4
    kk = []
    for e in (h, -h):
        v = torch.ones(nx * ny, dtype=torch.float64, device="cuda")
        v[c] += e
        kk.append(s.solve(o, sigma=v)["kappa"])
    assert abs((kk[0] - kk[1]) / (2 * h) - g[c]) <= 1e-6 * np.abs(g).max()
