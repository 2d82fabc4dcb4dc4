"""A batch of one, two, four and more orders: the operators run side by side
in a captured FP64 iteration; each slot's result is that of the solve alone."""
import pytest
import torch

import seeded_inputs as SI

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("orders", [(7,), (5, 7), (3, 4, 6, 8), (2, 3, 4, 5, 6, 7, 9)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_orders_share_a_batch(semlib, orders, precision):
    print(f"case: batch of orders {orders} {precision}", flush=True)
    meshes = [semlib.box_mesh(N, (4, 3, 2), vertices=SI.jittered_box_vertices((4, 3, 2), seed=N), with_fp32=True)
              for N in orders]
    bs = [m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, 4)).cuda()) for m in meshes]
    B = semlib.Batch(max_slots=8)
    runs = [B.solve(meshes, bs, tol=1e-10, precision=precision) for _ in range(3)]  # the graph replayed
    for m, b, *got in zip(meshes, bs, *(xs for xs, _ in runs)):
        (alone,), (r,) = B.solve([m], [b], tol=1e-10, precision=precision)
        assert r.ok and all(torch.equal(x, alone) for x in got)
    # the same without graphs
    xs, res = B.solve(meshes, bs, tol=1e-10, precision=precision, use_graph=False)
    assert all(r.ok for r in res) and all(torch.equal(x, y) for x, y in zip(xs, runs[0][0]))
    B.close()
    for m in meshes:
        m.close()
