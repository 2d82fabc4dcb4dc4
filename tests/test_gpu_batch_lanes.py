"""Batches whose operators run side by side, in turn, or change from one to the
other as slots converge: each slot's result is that of the solve alone."""
import pytest
import torch

import seeded_inputs as SI

pytestmark = pytest.mark.gpu


# three orders that share the device, the same beside smaller slots that
# converge first and larger ones that fill it, nine orders of a few elements
@pytest.mark.parametrize("specs", [
    [(5, (6, 6, 6)), (7, (6, 6, 6)), (9, (6, 6, 6))],
    [(5, (6, 6, 6)), (7, (6, 6, 6)), (9, (6, 6, 6)), (5, (2, 2, 2)), (9, (2, 1, 2)), (7, (12, 12, 13))],
    [(N, (2, 2, 2)) for N in range(2, 11)]])
@pytest.mark.parametrize("coarse", [False, True])
def test_side_by_side_and_back(semlib, specs, coarse):
    print(f"case: batch lanes {specs} coarse={coarse}", flush=True)
    meshes = [semlib.box_mesh(N, nel, vertices=SI.jittered_box_vertices(nel, seed=N)) for N, nel in specs]
    if coarse:
        for m in meshes[::2]:
            m.set_coarse(4, 0.05)
    bs = [m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, 4)).cuda()) for m in meshes]
    B = semlib.Batch(max_slots=len(specs))
    runs = [B.solve(meshes, bs, tol=1e-10) for _ in range(3)]  # the graphs replayed
    plain, _ = B.solve(meshes, bs, tol=1e-10, use_graph=False)
    for m, b, y, *got in zip(meshes, bs, plain, *(xs for xs, _ in runs)):
        (alone,), (r,) = B.solve([m], [b], tol=1e-10)
        assert r.ok and torch.equal(y, alone) and all(torch.equal(x, alone) for x in got)
    B.close()
    for m in meshes:
        m.close()
