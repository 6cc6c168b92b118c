"""The limit of obte_solve_noalloc: what it admitted when workspaces held the
pass inputs by cell it still admits, one system more it refuses; and where rows
along y make the wrap inflow too long it sweeps with rows along x."""
import numpy as np
import pytest
import torch

from inputs import gen
from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu
LIMIT = 32 << 20


@pytest.fixture(scope="module")
def P():
    return require_gpu()


def _align(n):
    return (n + 255) // 256 * 256


def _solver(P, n, n_mfp):
    """Two directions and n_mfp MFPs on a pore-free cell."""
    d3 = len(n) == 3
    s = 0.6 ** 0.5, 0.3 ** 0.5, 0.1 ** 0.5
    dirs = np.array([s, [-v for v in s]]) if d3 else np.array([[0.8, 0.6], [-0.8, -0.6]])
    return P.Solver(ndim=len(n), n=n, L=(1e-7, 1e-7, 1e-7)[:len(n)], solid=np.ones(int(np.prod(n)), np.uint8),
                    periodic=(1, 1, 0), grad_axis=0, dT=1.0, mfp=np.logspace(-9, -6, n_mfp), dirs=dirs,
                    dir_w=[0.5, 0.5], kappa_m=np.full(n_mfp, 1.0 / n_mfp))


def _noalloc(P, s, o):
    T = torch.empty(s.n_cells, dtype=torch.float64, device="cuda")
    st = P.obte.obte_solve_noalloc(s.mesh, o, None, stream=s.stream, T_L=T)
    torch.cuda.synchronize()
    return st.as_dict(), T


def _bytes(P, n, n_mfp):
    s = _solver(P, n, n_mfp)
    return P.obte.obte_workspace_size(s.mesh, s.opts())


def _last(size, lo, hi):
    """The largest n with size(n) <= LIMIT."""
    assert size(lo) <= LIMIT < size(hi)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if size(mid) <= LIMIT else (lo, mid)
    return lo


# W: systems per workgroup, for the work items' 20 bytes (16 at the time)
@pytest.mark.parametrize("n,W", [((8, 8, 4), 1), ((9, 5, 3), 1)])
def test_admits_what_it_did_3d(P, n, W):
    nx, ny, nz = n
    nc = nx * ny * nz
    row = (nx * 68 + 15) // 16 * 16
    tables = _align(2 * (ny * nz + 4) * row) - _align(7 * nc * 8)

    def size(k):
        s = _solver(P, n, k)
        items = 2 * ((k + W - 1) // W)
        now = P.obte.obte_workspace_size(s.mesh, s.opts())
        return now - tables - (_align(20 * items) - _align(16 * items))

    k = _last(size, 500, 20000)
    s = _solver(P, n, k)
    o = s.opts(outer_tol=0.0, max_outer=2)
    assert P.obte.obte_workspace_size(s.mesh, o) > LIMIT
    st, T = _noalloc(P, s, o)
    ref = s.solve(o)
    assert st["kappa"] == ref["kappa"] and torch.equal(T, ref["T_L"])
    over = _solver(P, n, k + 1)
    with pytest.raises(P.ObteError) as e:
        _noalloc(P, over, o)
    assert e.value.status == P.obte.OBTE_ERR_NOMEM


def test_rows_along_x_where_the_inflow_is_too_long(P):
    n = (40, 80)
    # the wrap inflow of 80 values for 40 a system: 40 x 16 bytes a system
    k = _last(lambda q: _bytes(P, n, q), 20, 2000)
    s = _solver(P, n, k + 1)
    o = s.opts(outer_tol=1e-11, inner_tol=1e-13, max_outer=500)
    assert LIMIT < P.obte.obte_workspace_size(s.mesh, o) < LIMIT + 2 * k * 40 * 16
    st, T = _noalloc(P, s, o)
    ref = s.solve(o)
    # another sweep order: the same fixed point to the outer tolerance
    assert st["status"] == 0 and ref["status"] == 0
    assert abs(st["kappa"] - ref["kappa"]) <= 1e-9 * ref["kappa"]
    assert float((T - ref["T_L"]).abs().max()) <= 1e-8 * float(ref["T_L"].abs().max())


def test_admits_what_the_query_says(P):
    n = (33, 21)
    k = _last(lambda q: _bytes(P, n, q), 20, 5000)
    assert P.obte.obte_noalloc_scratch_bytes() == LIMIT
    s = _solver(P, n, k)
    st, _ = _noalloc(P, s, s.opts(outer_tol=0.0, max_outer=1))
    assert st["outer_iters"] == 1
