"""A resident run that is called off leaves everything as it was, and the
general iteration goes on from there: the bits, iteration counts and statuses
of a solve that never took a resident run.  The call-off is forced from the
host (a wait of 0: no run stands); every kernel ends normally, its workgroups
giving up at the first exchange that is not complete, or, where there is one
workgroup, doing the whole run for nothing."""
import pytest
import torch

import seeded_inputs as SI

pytestmark = pytest.mark.gpu

# one workgroup (the run is completed and then discarded), several, one more
# than the compute units (two elements each), factors read every iteration
CASES = [(3, (1, 1, 1)), (5, (2, 3, 2)), (7, (1, 1, 257)), (9, (9, 8, 8)), (10, (4, 4, 5))]


def _same(a, b):
    return torch.equal(a.view(torch.int64), b.view(torch.int64))


@pytest.mark.parametrize("N,nel", CASES)
def test_called_off_run_changes_nothing(semlib, N, nel):
    print(f"case: resident call-off N={N} nel={nel}", flush=True)
    m = semlib.box_mesh(N, nel, vertices=SI.jittered_box_vertices(nel, seed=N), with_fp32=True)
    b = m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, 3)).cuda())
    guess = m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, 4)).cuda())
    solves = [dict(fixed_iters=4), dict(fixed_iters=40), dict(tol=1e-10, max_iter=20000),
              dict(tol=1e-10, max_iter=20000, precision="mixed"), dict(tol=1e-10, max_iter=5, raise_on_error=False),
              dict(tol=1e-10, max_iter=20000, use_graph=False, poll_every=5)]
    m.set_resident(False)
    assert not m.resident_info()["in_use"]
    want = [m.solve(b, guess.clone(), **kw) for kw in solves]
    assert m.resident_info() == {"in_use": False, "runs": 0, "called_off": 0}
    m.set_resident(True, 0.0)
    assert m.resident_info()["in_use"]
    for kw, (xw, rw) in zip(solves, want):
        before = m.resident_info()["called_off"]
        x, r = m.solve(b, guess.clone(), **kw)
        assert m.resident_info()["called_off"] > before and m.resident_info()["runs"] == 0, kw
        assert _same(x, xw), kw
        assert (r.status, r.iterations, r.outer_iterations) == (rw.status, rw.iterations, rw.outer_iterations), kw
    # the mesh takes resident runs again as if none had been called off
    m.set_resident(True)
    ref = semlib.box_mesh(N, nel, vertices=SI.jittered_box_vertices(nel, seed=N), with_fp32=True)
    for kw in solves:
        x, r = m.solve(b, guess.clone(), **kw)
        xr, rr = ref.solve(b, guess.clone(), **kw)
        assert _same(x, xr) and r.iterations == rr.iterations, kw
    assert m.resident_info()["runs"] == ref.resident_info()["runs"] > 0
    assert ref.resident_info()["called_off"] == 0
    ref.close()
    m.close()


def test_called_off_once_a_solve(semlib):
    """A solve whose run was called off does not try again at each of its
    restarts and refinement steps: every try costs the wait."""
    print("case: resident tries of one solve", flush=True)
    m = semlib.box_mesh(5, (4, 4, 4), vertices=SI.jittered_box_vertices((4, 4, 4), seed=5), with_fp32=True)
    b = m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, 3)).cuda())
    m.set_resident(True, 0.0)
    tries = 0
    for precision in ("fp64", "mixed"):
        x, r = m.solve(b, tol=1e-12, max_iter=20000, precision=precision, inner_tol=1e-2, raise_on_error=False)
        if precision == "mixed":
            assert r.outer_iterations >= 3
        tries += 1
        assert m.resident_info()["called_off"] == tries, (precision, r.outer_iterations)
    m.close()


def test_resident_config_is_checked(semlib):
    m = semlib.box_mesh(3, (2, 2, 2))
    for enable, wait in ((2, 1.0), (-1, 1.0), (1, 1001.0), (1, float("nan"))):
        assert m._lib.sem_set_resident_config(m._h, enable, wait) == 1
    assert m.resident_info()["in_use"]
    m.set_coarse(4)
    assert not m.resident_info()["in_use"]
    m.close()
