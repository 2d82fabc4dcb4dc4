"""CG iterations whose gather-scatter also sums p.Ap (lattice meshes) against
the two launches of the plan: the same sums in the same order, the same bits."""
import pytest
import torch

import seeded_inputs as SI

pytestmark = pytest.mark.gpu


# fewer partials than threads, a few, and more than the workgroup's first round
@pytest.mark.parametrize("N,nel,periodic", [(1, (5, 4, 3), (0, 0, 0)), (2, (2, 3, 2), (1, 0, 1)),
                                            (5, (1, 4, 3), (0, 0, 1)), (7, (11, 12, 10), (0, 1, 0)),
                                            (12, (2, 1, 2), (1, 0, 0))])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_sum_beside_the_gather_scatter(semlib, N, nel, periodic, precision):
    print(f"case: gs + sigma N={N} nel={nel} periodic={periodic} {precision}", flush=True)
    m = semlib.box_mesh(N, nel, periodic=periodic, with_fp32=True)
    m.set_coarse(4, 0.05)
    b = m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, seed=9)).cuda())
    out = []
    for kind in ("plan", "auto", "plan"):
        m.set_gs_kind(kind)
        x, res = m.solve(b, tol=1e-9, max_iter=400, precision=precision)
        out.append((x.clone(), res.iterations, res.ok))
    assert out[0][2]
    for x, its, ok in out[1:]:
        assert its == out[0][1] and torch.equal(x, out[0][0])
    m.close()
