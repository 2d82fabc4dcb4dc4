"""Solves on a device that runs out of memory (CPU: fake_hip.cpp): whichever
allocation of a solve fails, that call and every later one work on memory that
is there."""
import pytest

import fakehip


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fakehip.build(tmp_path_factory.mktemp("fakehip"))


# the mesh of 8 elements takes the resident run: its scratch is not needed by
# the general iteration, which a mesh without room for it goes on with
def test_resident_scratch(runtime):
    out = fakehip.run(runtime, """
        # the solve vectors first (profiled solves keep to the general iteration)
        for nth in range(3):
            m, info = mesh(4, (2, 2, 2), fp32=True)
            b, x = np.ones(info.n_local), np.zeros(info.n_local)
            o = opts(fixed_iters=4, use_graph=0, profile=1)
            L.check(lib.sem_pcg_solve(m, b.ctypes.data, x.ctypes.data, C.byref(o), None, None), "solve")
            assert not launches("resident_kernel")
            o = opts(fixed_iters=4, use_graph=0)
            fake.fake_fail_in(nth)
            st = lib.sem_pcg_solve(m, b.ctypes.data, x.ctypes.data, C.byref(o), None, None)
            fake.fake_fail_in(-1)
            assert st == L.SEM_OK, (nth, st)
            fake.fake_clear()
            for _ in range(2):
                st = lib.sem_pcg_solve(m, b.ctypes.data, x.ctypes.data, C.byref(o), None, None)
                assert st == L.SEM_OK, (nth, st)
            runs = launches("resident_kernel")
            assert len(runs) == 2 and all(fake.fake_has_scratch(i) for i in runs), (nth, runs)
            fake.fake_clear()
            lib.sem_free(m)
        assert fake.fake_null_uses() == 0
        print("done")
        """)
    assert "done" in out


def test_error_ends_with_its_call(runtime):
    """A call that ran out of memory, at whichever of its allocations, leaves
    no error behind for the next."""
    fakehip.run(runtime, """
        m, info = mesh(3, (2, 2, 2))
        u, w = np.ones(info.n_local), np.zeros(info.n_local)
        def axgs():
            st = lib.sem_set_axgs_config(m, 1, 0, 0)
            return st or lib.sem_axgs(m, 0, u.ctypes.data, w.ctypes.data, None)
        def proj():
            p = C.c_void_p()
            st = lib.sem_proj_create(m, 2, C.byref(p))
            lib.sem_proj_free(p)
            return st
        calls = [axgs, proj, lambda: lib.sem_set_helmholtz(m, u.ctypes.data, u.ctypes.data, None),
                 lambda: lib.sem_set_schwarz(m, 1, None)]
        for c, call in enumerate(calls):
            refused = 0
            for nth in range(100):
                fake.fake_fail_in(nth)
                st = call()
                fake.fake_fail_in(-1)
                lib.sem_set_axgs_config(m, 0, 0, 0)
                assert lib.sem_ax(m, 0, u.ctypes.data, w.ctypes.data, None, None) == L.SEM_OK, (c, nth)
                if st == L.SEM_OK:
                    break
                assert st == L.SEM_ENOMEM, (c, nth, st)
                refused += 1
            assert refused > 0, c
        """)


def test_work_vectors(runtime):
    """Whichever work vector of a first solve, or coefficient of a first
    Helmholtz form, is refused: the next call has all of them."""
    fakehip.run(runtime, """
        def call(m, info, kind):
            b, x = np.ones(info.n_local), np.zeros(info.n_local)
            if kind == "helmholtz":
                return lib.sem_set_helmholtz(m, b.ctypes.data, b.ctypes.data, None)
            o = opts(fixed_iters=2, use_graph=0, profile=1)
            if kind == "mixed":
                o = opts(precision=L.SEM_PREC_MIXED, profile=1)
            return lib.sem_pcg_solve(m, b.ctypes.data, x.ctypes.data, C.byref(o), None, None)
        for kind, refusals in (("fp64", 4), ("mixed", 8), ("helmholtz", 5)):
            for nth in range(refusals):
                m, info = mesh(3, (2, 2, 2), fp32=True)
                fake.fake_fail_in(nth)
                assert call(m, info, kind) == L.SEM_ENOMEM, (kind, nth)
                fake.fake_fail_in(-1)
                assert call(m, info, kind) == L.SEM_OK, (kind, nth)
                assert fake.fake_null_uses() == 0, (kind, nth)
                lib.sem_free(m)
        """)
