"""The general CG iteration of small meshes (resident runs off), bit for bit:
every gather-scatter kind, captured and plain launches, and how often the host
polls, in FP64 and mixed precision, give the same iterate."""
import pytest
import torch

import seeded_inputs as SI

pytestmark = pytest.mark.gpu


def _bits(x):
    return x.view(torch.int64)


# orders with and without the update that sums the copies of w itself (N >= 3),
# the pipe map, periodic axes, free faces
@pytest.mark.parametrize("N,nel,periodic,faces,pipe", [
    (2, (5, 4, 3), (0, 0, 0), -1, False), (3, (4, 3, 5), (0, 1, 0), -1, False), (5, (3, 4, 2), (0, 0, 0), 0b010110, False),
    (7, (4, 4, 4), (0, 0, 0), -1, False), (7, (6, 6, 4), (0, 0, 1), -1, True), (9, (2, 3, 2), (1, 0, 0), -1, False)])
def test_kinds_and_launches_give_the_same_bits(semlib, N, nel, periodic, faces, pipe):
    print(f"case: general iteration N={N} nel={nel}", flush=True)
    if pipe:
        m = semlib.pipe_mesh(*nel, N=N, with_fp32=True)
    else:
        V = None if any(periodic) else SI.jittered_box_vertices(nel, seed=N)
        m = semlib.box_mesh(N, nel, vertices=V, periodic=periodic, dirichlet_faces=faces, with_fp32=True)
    b = m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, 3)).cuda())
    m.set_resident(False)
    for solve in (dict(tol=1e-10, max_iter=20000), dict(tol=1e-10, max_iter=20000, precision="mixed"),
                  dict(fixed_iters=37)):
        want, r0 = m.solve(b, **solve)
        for kind in ("auto", "plan", "stream"):
            m.set_gs_kind(kind)
            for launches in (dict(use_graph=True), dict(use_graph=False), dict(use_graph=True, poll_every=5),
                             dict(profile=True)):
                x, r = m.solve(b, **solve, **launches)
                assert torch.equal(_bits(x), _bits(want)), (solve, kind, launches)
                assert (r.iterations, r.outer_iterations) == (r0.iterations, r0.outer_iterations)
        m.set_gs_kind("auto")
    info = m.resident_info()
    assert not info["in_use"] and info["runs"] == 0 and info["called_off"] == 0
    m.close()


def test_resident_runs_stand(semlib):
    """With the default setting the same solves do take resident runs."""
    m = semlib.box_mesh(7, (4, 4, 4), vertices=SI.jittered_box_vertices((4, 4, 4), seed=7), with_fp32=True)
    b = m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, 3)).cuda())
    runs = 0
    for solve in (dict(tol=1e-10, max_iter=20000), dict(tol=1e-10, max_iter=20000, precision="mixed"),
                  dict(fixed_iters=37)):
        m.solve(b, **solve)
        info = m.resident_info()
        assert info["in_use"] and info["runs"] > runs and info["called_off"] == 0
        runs = info["runs"]
    m.close()
