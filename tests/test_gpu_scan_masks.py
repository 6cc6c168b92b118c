"""The row scan's masks, formed from the open cells of a row: pores scattered
over every lane, so that a row is closed at the start, the middle and the end of
each group of 1, 2, 4, 8, 16 and 32 lanes, for one to four cells per lane, with
and without padding, in both row orientations and in 3D; pass for pass against
the oracle."""
import dataclasses

import numpy as np
import pytest

from inputs import gen
from oracle.bte import Problem, source_iteration
from tests.gpu_common import gpu_solve, oracle_full, rel, require_gpu

pytestmark = pytest.mark.gpu
NM = 1e-9


@pytest.fixture(scope="module")
def P():
    return require_gpu()


def _pores(shape, seed):
    """One cell in twelve is a pore; a row without any and a closed one stay."""
    rng = np.random.default_rng(seed)
    s = (rng.random(shape) > 1 / 12).astype(np.uint8)
    s[..., 1, :] = 1
    s[..., -2, : shape[-1] // 2] = 0
    # a cell between pores has no equation for its temperature
    s &= np.roll(s, 1, -1) | np.roll(s, -1, -1) | np.roll(s, 1, -2) | np.roll(s, -1, -2)
    return s


def _check(P, w):
    prob = Problem(w)
    K = 3
    ref = source_iteration(prob, n_passes=K)
    # bars of the lockstep tests: FP64 rounding over K passes, FP32 likewise
    for prec, tol, bar in ((0, 1e-14, 1e-10), (1, 1e-6, 1e-4)):
        r = gpu_solve(P, w, precision=prec, outer_tol=0.0, max_outer=K, inner_tol=tol, fourier_tol=1e-14, max_inner=400)
        assert r["outer_iters"] == K
        assert abs(r["kappa"] - ref["kappa_cc"]) <= bar * abs(ref["kappa_cc"]), prec
        assert rel(r["T_L"], oracle_full(prob, ref["T_L"])) < bar, prec


# full and padded rows of one to four cells per lane along x; along y (the last two)
@pytest.mark.parametrize("nx,ny", [(64, 12), (51, 12), (128, 10), (99, 9), (192, 8), (150, 8), (256, 6), (201, 6),
                                   (40, 100), (70, 200)])
def test_scattered_pores(P, nx, ny):
    _check(P, gen.small_2d(nx, ny, solid=_pores((ny, nx), [nx, ny]), n_dir=8, n_mfp=2, mfp_lo=50 * NM, mfp_hi=5e-6,
                           L=100 * NM))


@pytest.mark.parametrize("nx,ny,nz", [(64, 4, 3), (51, 4, 3), (128, 4, 2), (150, 4, 2), (192, 4, 2), (201, 4, 2),
                                      (256, 4, 2)])
def test_scattered_pores_3d(P, nx, ny, nz):
    w = gen.small_3d(nx, ny, nz, solid=_pores((nz, ny, nx), [nx, ny, nz]), n_theta=2, n_phi=4, n_mfp=2)
    _check(P, dataclasses.replace(w, grad_axis=1))
