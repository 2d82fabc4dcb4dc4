"""The assembly of the Schwarz local solves takes a lane per node on small
meshes and a lane per column on larger ones: on boxes of unit cubes, periodic
in all directions, the preconditioner of a larger box repeats that of one
period, whichever form each takes."""
import numpy as np
import pytest
import torch

import seeded_inputs as SI

pytestmark = pytest.mark.gpu


def _unit_cubes(semlib, N, nel):
    z, y, x = np.meshgrid(*[np.arange(n + 1, dtype=np.float64) for n in nel[::-1]], indexing="ij")
    return semlib.box_mesh(N, nel, vertices=np.stack([x, y, z], axis=-1).reshape(-1, 3), periodic=(1, 1, 1))


# workgroups of columns: 32 and 256, 21 and 168, 128 and 256, 32 and 256, 54 and
# 216, 96 and 288
@pytest.mark.parametrize("N,nel,times", [(3, (8, 8, 8), (2, 2, 2)), (4, (5, 7, 6), (2, 2, 2)), (3, (8, 16, 16), (2, 1, 1)),
                                         (7, (4, 4, 8), (2, 2, 2)), (7, (6, 6, 6), (1, 2, 2)), (12, (4, 4, 6), (1, 1, 3))])
@pytest.mark.parametrize("coarse", [0, 4])
def test_larger_boxes_repeat_a_period(semlib, N, nel, times, coarse):
    print(f"case: schwarz assembly N={N} nel={nel} times={times} coarse={coarse}", flush=True)
    big = tuple(a * b for a, b in zip(nel, times))
    s, m = _unit_cubes(semlib, N, nel), _unit_cubes(semlib, N, big)
    P3 = (N + 1) ** 3
    e = torch.arange(m.E, device="cuda")
    ex, ey, ez = e % big[0], e // big[0] % big[1], e // (big[0] * big[1])
    period = ex % nel[0] + nel[0] * (ey % nel[1] + nel[1] * (ez % nel[2]))
    r = s.scatter(torch.from_numpy(SI.uniform_global_values(s.n_global, seed=N)).cuda())
    for q in (s, m):
        q.set_schwarz(True)
        if coarse:
            q.set_coarse(coarse, 0.05)
    ref = s.precond(r).view(-1, P3)[period].reshape(-1)
    z = m.precond(r.view(-1, P3)[period].reshape(-1).contiguous())
    # the local problems are those of one period up to the rounding of the
    # element edge lengths (integers here: none); the coarse interval is a row sum
    assert (z - ref).abs().max() <= 1e-13 * ref.abs().max()
    s.close()
    m.close()
