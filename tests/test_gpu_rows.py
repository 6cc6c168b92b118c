"""The 2D sweep's two row orientations, the 3D sweep's row order and the masked
row scan, pass for pass against the oracle: rows that fill the wave exactly, rows padded by one to
three cells, a few cells only, meshes where rows along y are wider or are not
taken, pores on the boundary, both gradient axes, with and without a sigma
field; and checkpoints written before rows along y existed."""
import dataclasses
import struct

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


def _mask(nx, ny):
    s = np.ones((ny, nx), np.uint8)
    s[ny // 3: ny // 3 + max(1, ny // 4), nx // 4: nx // 4 + max(1, nx // 3)] = 0
    if nx > 4 and ny > 4:
        s[0, nx // 2] = 0
        s[ny // 2, 0] = 0
        s[-1, -1] = 0
    return s


# (nx, ny): full lanes for one and two cells per lane; padding of 1 to 3;
# staged batches cut short (ny, nx not multiples of 8 or 4); few rows; rows
# along y wider than along x; rows along y too wide to be taken
SHAPES = [(64, 64), (128, 128), (65, 63), (3, 5), (5, 3), (2, 7), (129, 30), (30, 129), (40, 128), (100, 130),
          (33, 34), (190, 197), (70, 9)]


@pytest.mark.parametrize("nx,ny", SHAPES)
@pytest.mark.parametrize("sigma", [False, True])
def test_rows_lockstep(P, nx, ny, sigma):
    rng = np.random.default_rng([nx, ny])
    sg = 2.0 ** rng.uniform(-1, 1, nx * ny) if sigma else None
    w = gen.small_2d(nx, ny, solid=_mask(nx, ny), n_dir=12, n_mfp=2, mfp_lo=50 * NM, mfp_hi=5e-6, L=100 * NM,
                     grad_axis=int(sigma), sigma=sg)
    prob = Problem(w)
    K = 4
    ref = source_iteration(prob, n_passes=K)
    Jref = np.zeros((w.n_cells, 2))
    Jref[prob.mesh.cells] = ref["J"]
    for prec, tol, bar in ((0, 1e-14, 1e-10), (1, 1e-6, 1e-4)):
        r = gpu_solve(P, w, precision=prec, outer_tol=0.0, max_outer=K, inner_tol=tol, fourier_tol=1e-14,
                      max_inner=400)
        assert r["outer_iters"] == K
        assert abs(r["kappa"] - ref["kappa_cc"]) <= bar * abs(ref["kappa_cc"]), prec
        assert abs(r["kappa_face"] - ref["kappa_face"]) <= bar * abs(ref["kappa_face"]), prec
        assert rel(r["T_L"], oracle_full(prob, ref["T_L"])) < bar, prec
        assert rel(r["J"], Jref) < bar, prec


# 3D: full lanes, padding, three cells per lane, the fewest planes, y rows
# that leave one or two rows over the unrolled ones
SHAPES3 = [(64, 5, 3), (65, 4, 2), (130, 3, 2), (3, 3, 2), (9, 7, 5), (20, 6, 4)]


@pytest.mark.parametrize("nx,ny,nz", SHAPES3)
@pytest.mark.parametrize("sigma", [False, True])
def test_rows_lockstep_3d(P, nx, ny, nz, sigma):
    rng = np.random.default_rng([nx, ny, nz])
    sg = 2.0 ** rng.uniform(-1, 1, nx * ny * nz) if sigma else None
    s = np.ones((nz, ny, nx), np.uint8)
    s[:, ny // 3, nx // 4: nx // 4 + max(1, nx // 3)] = 0
    s[0, -1, 0] = 0
    w = gen.small_3d(nx, ny, nz, solid=s, n_theta=4, n_phi=6, n_mfp=2, sigma=sg)
    w = dataclasses.replace(w, grad_axis=int(sigma))
    prob = Problem(w)
    K = 4
    ref = source_iteration(prob, n_passes=K)
    Jref = np.zeros((w.n_cells, 3))
    Jref[prob.mesh.cells] = ref["J"]
    for prec, tol, bar in ((0, 1e-14, 1e-10), (1, 1e-6, 1e-4)):
        r = gpu_solve(P, w, precision=prec, outer_tol=0.0, max_outer=K, inner_tol=tol, fourier_tol=1e-14,
                      max_inner=400)
        assert r["outer_iters"] == K
        assert abs(r["kappa"] - ref["kappa_cc"]) <= bar * abs(ref["kappa_cc"]), prec
        assert abs(r["kappa_face"] - ref["kappa_face"]) <= bar * abs(ref["kappa_face"]), prec
        assert rel(r["T_L"], oracle_full(prob, ref["T_L"])) < bar, prec
        assert rel(r["J"], Jref) < bar, prec


def test_wide_group_with_wider_rows_along_y(P):
    """Eight FP64 systems per workgroup were accepted for nx <= 128 whatever
    ny: they still are where rows along y need three cells per lane."""
    w = gen.small_2d(128, 140, solid=_mask(128, 140), n_dir=8, n_mfp=8, L=100 * NM)
    a = gpu_solve(P, w, want_J=False, outer_tol=1e-9, waves_per_group=8)
    b = gpu_solve(P, w, want_J=False, outer_tol=1e-9, waves_per_group=1)
    assert a["kappa"] == b["kappa"] and np.array_equal(a["T_L"], b["T_L"])


@pytest.mark.parametrize("prec", [0, 1])
def test_checkpoint_of_rows_along_x_only(P, prec, tmp_path):
    """A file in the earlier form (wrap inflows of rows along x for every
    system, in units of the inflow) loads, and the resumed solve ends where
    the uninterrupted one does."""
    nx, ny = 14, 17
    w = gen.small_2d(nx, ny, solid=_mask(nx, ny), n_dir=8, n_mfp=3)
    opt = dict(precision=prec, outer_tol=1e-10 if prec == 0 else 1e-7, inner_tol=1e-13 if prec == 0 else 1e-6,
               max_outer=5000)
    full = gpu_solve(P, w, want_J=False, **opt)
    r = gpu_solve(P, w, want_J=False, **dict(opt, max_outer=6))
    s = r["solver"]
    new, old = str(tmp_path / "new"), str(tmp_path / "old")
    s.checkpoint_save(new)
    raw = open(new, "rb").read()
    hdr = list(struct.unpack("9i", raw[:36]))
    wrap = hdr[4]
    assert wrap == max(nx, ny)
    t = np.float64 if prec == 0 else np.float32
    nw = s.n_walls
    at = 36 + 8 * 4 + 8 * nx * ny * 3 + 16 * nw                     # ctrl, T_L, sT (2), Tw (2)
    n = s.n_systems * wrap * t().itemsize
    U = np.frombuffer(raw[at:at + n], t).reshape(s.n_systems, wrap)
    c = (w.mfp[:, None] * np.abs(w.dirs[None, :, 1]) / (w.L[1] / ny)).reshape(-1, 1)
    hdr[0], hdr[4] = 0x4f425447, nx
    body = np.ascontiguousarray((U[:, :nx] * c).astype(t)).tobytes()
    open(old, "wb").write(struct.pack("9i", *hdr) + raw[36:at] + body + raw[at + n:])
    s2 = P.Solver.from_workload(w)
    o = s2.opts(**dict(opt, init=1))
    s2.ensure_workspace(o)
    s2.checkpoint_load(old)
    out = s2.solve(o, want_T_L=True)
    assert out["status"] == 0 and out["outer_iters"] > 6
    assert abs(out["kappa"] - full["kappa"]) <= (1e-8 if prec == 0 else 1e-4) * full["kappa"]
