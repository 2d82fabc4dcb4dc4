"""Host side of the resident CG on the CPU (fake_hip.cpp): how many iterations
a launch takes, and which runs of several threads are in flight together."""
import pytest

import fakehip


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fakehip.build(tmp_path_factory.mktemp("fakehip"))


def test_iterations_of_a_launch(runtime):
    """A launch holds its compute units for some milliseconds, well below the
    20 ms that another process's run waits for them: 512 iterations with the
    factors on chip, fewer where they are read every iteration."""
    fakehip.run(runtime, """
        fake.fake_set_verdict(1)
        cases = [(4, (2, 2, 2), [512, 88]), (9, (11, 11, 10), [128] * 4 + [88]), (7, (13, 13, 12), [256] * 2 + [88]),
                 (4, (16, 16, 20), [512, 88])]
        for N, nel, want in cases:
            m, info = mesh(N, nel)
            b, x = np.ones(info.n_local), np.zeros(info.n_local)
            o = opts(fixed_iters=600)
            fake.fake_clear()
            L.check(lib.sem_pcg_solve(m, b.ctypes.data, x.ctypes.data, C.byref(o), None, None), "solve")
            got = [fake.fake_iters(i) for i in launches("resident_kernel")]
            assert got == want, (N, nel, got)
            lib.sem_free(m)
        """)


def test_short_solves_take_the_general_iteration(runtime):
    """Below four iterations a run costs more than it saves."""
    fakehip.run(runtime, """
        fake.fake_set_verdict(1)
        m, info = mesh(5, (3, 3, 3))
        b, x = np.ones(info.n_local), np.zeros(info.n_local)
        for steps, runs in ((1, 0), (3, 0), (4, 1), (5, 1)):
            o = opts(fixed_iters=steps, use_graph=0)
            fake.fake_clear()
            L.check(lib.sem_pcg_solve(m, b.ctypes.data, x.ctypes.data, C.byref(o), None, None), "solve")
            assert len(launches("resident_kernel")) == runs, steps
        """)


def test_runs_in_flight_fit_every_xcd(runtime):
    """The workgroups of a launch go to the 8 XCDs in turn, 32 compute units
    each: 129 and 127 workgroups fit the device's 256 but put 17 + 16 on one
    XCD, so one run waits for the other; 128 and 128 run side by side."""
    fakehip.run(runtime, """
        import threading
        fake.fake_set_verdict(1)
        fake.fake_hold_ms(300)
        def flight(sizes):
            ms = [mesh(3, nel) for nel in sizes]
            def work(m, info):
                b, x = np.ones(info.n_local), np.zeros(info.n_local)
                o = opts(fixed_iters=4)
                L.check(lib.sem_pcg_solve(m, b.ctypes.data, x.ctypes.data, C.byref(o), None, None), "solve")
            fake.fake_clear()
            th = [threading.Thread(target=work, args=m) for m in ms]
            for t in th:
                t.start()
            for t in th:
                t.join()
            assert len(launches("resident_kernel")) == len(sizes)
            return fake.fake_max_in_flight(), sorted(fake.fake_grid(i) for i in launches("resident_kernel"))
        assert flight([(1, 1, 257), (1, 1, 127)]) == (1, [127, 129])
        assert flight([(1, 1, 128), (1, 1, 128)]) == (2, [128, 128])
        assert flight([(1, 1, 64), (1, 1, 64), (1, 1, 56), (1, 1, 72)]) == (4, [56, 64, 64, 72])
        """)
