"""The resident CG of small meshes (one launch per run, every element on chip)
against the general iteration of the same library (profiled solves keep to
it): fixed-step iterates, whole FP64 and mixed solves, the limit and
restart paths, and solves that run at the same time on two streams."""
import threading

import numpy as np
import pytest
import torch

import seeded_inputs as SI

pytestmark = pytest.mark.gpu


def _mesh(semlib, N, nel, periodic=(0, 0, 0), **kw):
    V = SI.jittered_box_vertices(nel, seed=N)
    return semlib.box_mesh(N, nel, vertices=V, periodic=periodic, with_fp32=True, **kw)


def _rhs(m, seed):
    return m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, seed)).cuda())


# (N, elements, periodic): one workgroup, a ragged last workgroup (257 = 256 +
# 1, two elements per workgroup), the most elements with the factors on chip
# and the first with them read every iteration, every order's kernel, free
# faces and two-element periodic axes
CASES = [
    (3, (1, 1, 1), (0, 0, 0), None),
    (3, (2, 3, 2), (1, 0, 1), None),
    (7, (1, 1, 257), (0, 0, 1), None),
    (4, (16, 4, 4), (0, 1, 0), None),
    (5, (7, 6, 5), (0, 0, 0), 0b010110),
    (6, (9, 5, 6), (1, 0, 0), None),
    (7, (8, 8, 16), (0, 0, 1), None),      # 1,024: factors on chip
    (7, (5, 5, 41), (0, 0, 0), None),      # 1,025: read every iteration
    (8, (3, 5, 7), (0, 0, 0), None),
    (9, (2, 2, 2), (1, 1, 0), None),
    (9, (9, 8, 8), (0, 0, 0), None),
    (10, (4, 4, 5), (0, 0, 1), None),
]


@pytest.mark.parametrize("N,nel,periodic,faces", CASES)
def test_resident_matches_general(semlib, N, nel, periodic, faces):
    print(f"case: resident N={N} nel={nel} periodic={periodic}", flush=True)
    kw = {} if faces is None else {"dirichlet_faces": faces}
    m = _mesh(semlib, N, nel, periodic, **kw)
    b = _rhs(m, 3)
    for steps in (1, 2, 7):
        xr, rr = m.solve(b, fixed_iters=steps)
        xg, rg = m.solve(b, fixed_iters=steps, profile=True)
        assert rr.iterations == rg.iterations == steps
        # the iterations differ only in the order in which the partial sums of
        # the dot products are added (n eps of their terms, a few steps deep)
        assert float((xr - xg).norm()) <= 1e-12 * float(xg.norm()), steps
    for precision in ("fp64", "mixed"):
        xr, rr = m.solve(b, tol=1e-10, max_iter=20000, precision=precision)
        xg, rg = m.solve(b, tol=1e-10, max_iter=20000, precision=precision, profile=True)
        assert rr.ok and rg.ok and rr.rel_residual <= 1e-10
        assert abs(rr.iterations - rg.iterations) <= 2 + 0.02 * rg.iterations, (precision, rr.iterations, rg.iterations)
    m.close()


def test_resident_limit_and_guess(semlib):
    """max_iter inside a run, then a restart from the iterate it left."""
    m = _mesh(semlib, 5, (4, 4, 4))
    b = _rhs(m, 5)
    x, r = m.solve(b, tol=1e-10, max_iter=20, raise_on_error=False)
    assert r.status == 4 and r.iterations == 20
    x, r2 = m.solve(b, x, tol=1e-10, max_iter=5000)
    assert r2.ok and r2.rel_residual <= 1e-10
    # more iterations than one launch holds, in pieces and at once
    xa, ra = m.solve(b, fixed_iters=600)
    assert ra.iterations == 600
    m.close()


def test_resident_on_two_streams(semlib):
    """Solves of two threads on two streams (their workgroups do not fit on the
    device together, so one run waits for the other): the bits of each alone."""
    meshes = [_mesh(semlib, 7, (6, 6, 6)), _mesh(semlib, 5, (6, 5, 7))]
    bs = [_rhs(m, 11 + q) for q, m in enumerate(meshes)]
    torch.cuda.synchronize()
    alone = [m.solve(b, tol=1e-10)[0].cpu() for m, b in zip(meshes, bs)]
    got = [[], []]

    def work(q):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(6):
                x, r = meshes[q].solve(bs[q], tol=1e-10)
                assert r.ok
                got[q].append(x.cpu())

    th = [threading.Thread(target=work, args=(q,)) for q in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join(60)
    for q in range(2):
        assert len(got[q]) == 6
        for x in got[q]:
            assert torch.equal(x, alone[q])
    for m in meshes:
        m.close()
