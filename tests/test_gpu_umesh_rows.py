"""GPU: the unstructured path's sweeps in rows and its sums in strands at the
sizes where they change form, against the oracle: several wrap slots per lane
(4 and 8), chunks of systems with and without a part past a multiple of eight,
rows narrower and wider than a level, and passes that find a wrap settled after
one that had to correct it.

Tolerance: every system solved to 1e-14 on both sides; the passes' contraction
keeps that below 1e-12, the bound is the 1e-10 of the other lockstep tests."""
import numpy as np
import pytest

from inputs import gen
from oracle.bte import source_iteration
from oracle.umesh import UProblem
from tests.gpu_common import rel, require_gpu

pytestmark = pytest.mark.gpu
NM = 1e-9

CASES = {
    # 320 systems: chunks of 20 = 16 in four strands + 4
    "strands_and_rest": lambda: gen.unstructured_2d(9, 8, amp=0.3, tri=True, seed=7, n_dir=16, n_mfp=20,
                                                    pores=[((45 * NM, 45 * NM), 24 * NM)]),
    # 384 systems: chunks of 24, no rest; quadrilaterals
    "strands_only": lambda: gen.unstructured_2d(8, 8, amp=0.25, tri=False, seed=8, n_dir=16, n_mfp=24, grad_axis=1,
                                                pores=[((50 * NM, 50 * NM), 22 * NM)]),
    # 136 and 264 periodic faces in a direction: 4 and 8 wrap slots per lane
    "wrap_4_tri": lambda: gen.unstructured_2d(130, 6, amp=0.2, tri=True, seed=9, n_dir=8, n_mfp=2, Ly=5 * NM,
                                              pores=[((50 * NM, 2.5 * NM), 1.4 * NM)]),
    "wrap_8_quad": lambda: gen.unstructured_2d(260, 4, amp=0.2, tri=False, seed=10, n_dir=8, n_mfp=2, Ly=2 * NM,
                                               pores=[((50 * NM, 1 * NM), 0.6 * NM)]),
    "wrap_8_tri": lambda: gen.unstructured_2d(4, 256, amp=0.2, tri=True, seed=11, n_dir=8, n_mfp=2, Ly=6400 * NM,
                                              pores=[((50 * NM, 3200 * NM), 35 * NM)]),
    # three cells wide: rows of a few cells
    "narrow": lambda: gen.unstructured_2d(3, 70, amp=0.0, tri=False, seed=12, n_dir=8, n_mfp=2,
                                              pores=[((50 * NM, 50 * NM), 20 * NM)]),
}


@pytest.fixture(scope="module")
def P():
    return require_gpu()


@pytest.mark.parametrize("name", list(CASES))
def test_lockstep_vs_oracle(P, name):
    w = CASES[name]()
    K = 3
    s = P.UMeshSolver.from_workload(w)
    o = s.opts(outer_tol=0.0, max_outer=K, inner_tol=1e-14, max_inner=300, fourier_tol=1e-13)
    r = s.solve(o, sigma=w.sigma)
    prob = UProblem(w)
    ref = source_iteration(prob, n_passes=K)
    assert abs(r["kappa"] - ref["kappa_cc"]) <= 1e-10 * abs(ref["kappa_cc"])
    assert abs(r["kappa_face"] - ref["kappa_face"]) <= 1e-10 * abs(ref["kappa_face"])
    full = np.zeros(prob.mesh.n_cells)
    full[prob.mesh.cells] = ref["T_L"]
    assert rel(r["T_L"].cpu().numpy(), full) <= 1e-10


def test_settled_wrap_after_a_correction(P):
    """With a forcing term that any start meets, no pass corrects the wrap; a
    first solve that corrects leaves nothing behind in the second."""
    w = CASES["strands_and_rest"]()
    s = P.UMeshSolver.from_workload(w)
    loose = dict(outer_tol=0.0, max_outer=6, inner_tol=1e-2, inner_rtol=0.9, max_inner=50, fourier_tol=1e-13)
    a = s.solve(s.opts(**loose))
    s.solve(s.opts(outer_tol=0.0, max_outer=3, inner_tol=1e-14, max_inner=300, fourier_tol=1e-13))
    b = s.solve(s.opts(**loose))
    assert a["kappa"] == b["kappa"] and np.array_equal(a["T_L"].cpu().numpy(), b["T_L"].cpu().numpy())
