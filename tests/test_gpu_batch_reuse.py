"""A batch slot that ends within one step (a breakdown) and is admitted again
before the next step is another solve: the work tables follow the admission,
with and without the coarse term, and its result is that of the solve alone."""
import numpy as np
import pytest
import torch

import seeded_inputs as SI

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coarse", [False, True])
def test_slot_reused_after_breakdown(semlib, coarse):
    # FP64: a mixed slot meets the NaN in its FP64 residual, before any CG
    print(f"case: slot reuse after breakdown coarse={coarse}", flush=True)
    meshes = []
    for N, nel in ((5, (3, 3, 2)), (7, (4, 3, 3))):
        m = semlib.box_mesh(N, nel, vertices=SI.jittered_box_vertices(nel, seed=N), with_fp32=True)
        if coarse:
            m.set_coarse(3, 0.05)
        meshes.append(m)
    b = meshes[1].scatter(torch.from_numpy(SI.uniform_global_values(meshes[1].n_global, 4)).cuda())
    B = semlib.Batch(max_slots=2)
    (alone,), _ = B.solve([meshes[1]], [b], tol=1e-10)
    bad = torch.full((meshes[0].n_local,), float("nan"), dtype=torch.float64, device="cuda")
    slot = B.admit(meshes[0], bad, tol=1e-10)
    for _ in range(4):
        B.step(8)
        if slot in B.finished():
            break
    assert slot in B.finished()
    _, r = B.retire(slot)
    assert r.status != 0
    assert B.admit(meshes[1], b, tol=1e-10) == slot
    while B.step(16):
        pass
    x, r = B.retire(slot)
    assert r.ok and torch.equal(x, alone)
    B.close()
    for m in meshes:
        m.close()
