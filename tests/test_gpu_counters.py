"""The iteration and sweep counters of a solve and of an adjoint do not depend
on what the workspace held, also where the systems' counters do not fill whole
256-byte units."""
import dataclasses

import numpy as np
import pytest

from inputs import gen
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu
NM = 1e-9


@pytest.fixture(scope="module")
def P():
    return require_gpu()


@pytest.mark.parametrize("n_dir,n_mfp", [(8, 3), (12, 5), (8, 4)])
def test_counters_on_a_used_workspace(P, n_dir, n_mfp):
    import torch
    nx, ny = 12, 10
    sg = 2.0 ** np.random.default_rng(1).uniform(-1, 1, nx * ny)
    w = dataclasses.replace(gen.small_2d(nx, ny, n_dir=n_dir, n_mfp=n_mfp, L=100 * NM), sigma=sg)
    got = []
    for fill in (0, 0x3f):
        s = P.Solver.from_workload(w)
        o = s.opts(outer_tol=1e-10, keep_state=1, max_outer=2000)
        s.ensure_workspace(o).fill_(fill)
        r = s.solve(o, sigma=w.sigma)
        its, sws = s.system_counts()
        assert r["inner_iters"] == its.sum() and r["sweeps"] == sws.sum()
        # a pass takes at least one sweep of a system, and two per iteration and two more at most
        assert np.all(sws >= r["outer_iters"]) and np.all(sws <= 2 * r["outer_iters"] + 2 * its)
        _, a = s.adjoint(o)
        torch.cuda.synchronize()
        got.append((r["inner_iters"], r["sweeps"], its.tolist(), sws.tolist(), a["inner_iters"], a["sweeps"]))
    assert got[0] == got[1]
