"""The fused preconditioner kernels at the edges of their ranges: M^-1 r with
the Schwarz local solves and the coarse term (element sums taken inside the
local solves, prolongation inside their assembly) and with Jacobi and the
coarse term, against the oracles.  Orders 3 (one plane of inner nodes) and 12
(the largest), element counts that leave the last workgroup of the column
kernels partly empty, single-element and two-element periodic axes, walls and
free faces meeting at an edge."""
import numpy as np
import pytest
import torch

import seeded_inputs as SI
from oracle.coarse import CoarseOracle
from oracle.schwarz import SchwarzOracle

pytestmark = pytest.mark.gpu

# the tolerances of test_gpu_schwarz.py and test_gpu_coarse.py: the local
# solves agree to a few thousand ulps of their condition, the rest to rounding
TOL_SCHWARZ, TOL_JACOBI = 1e-11, 1e-12

CASES = [
    (2, (3, 2, 5), (0, 0, 1), None),
    (3, (5, 3, 7), (0, 1, 0), None),
    (3, (1, 2, 3), (1, 1, 0), None),       # one periodic element: its own neighbour
    (6, (3, 1, 2), (0, 0, 1), None),       # 49 columns: a workgroup of five elements
    (8, (2, 3, 1), (0, 0, 0), 0b010010),   # walls and free faces
    (12, (2, 1, 2), (0, 0, 1), None),
]


@pytest.mark.parametrize("N,nel,periodic,dirichlet", CASES)
def test_precond_edges(semlib, oracle_mod, N, nel, periodic, dirichlet):
    print(f"case: precond edges N={N} nel={nel} periodic={periodic} dirichlet={dirichlet}", flush=True)
    V = SI.jittered_box_vertices(nel, seed=N)
    kw = {} if dirichlet is None else {"dirichlet_faces": dirichlet}
    m = semlib.box_mesh(N, nel, vertices=V, periodic=periodic, **kw)
    om = oracle_mod.OracleMesh(N, nel, vertices=V, periodic=periodic, dirichlet=dirichlet)
    live = om.local_mask() == 0
    r = SI.uniform_global_values(om.nglob, seed=17 * N)[om.numbering()] * live
    rd = torch.from_numpy(np.ascontiguousarray(r)).cuda()
    k, frac = 3, 0.05
    C = CoarseOracle(om, k=k, frac=frac)
    zs, zc = SchwarzOracle(om).apply(r), C.coarse(r)

    def check(ref, tol):
        z = m.precond(rd).cpu().numpy()
        assert np.linalg.norm(z - ref) <= tol * np.linalg.norm(ref)
        assert np.max(np.abs(z - ref)) <= tol * np.max(np.abs(ref))
        assert np.all(z[~live] == 0.0)

    m.set_schwarz(True)
    check(zs, TOL_SCHWARZ)
    m.set_coarse(k, frac)
    check(zs + zc, TOL_SCHWARZ)
    m.set_schwarz(False)
    check(C.inv * r + zc, TOL_JACOBI)
    m.close()
