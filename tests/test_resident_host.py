"""Host side of the resident CG on the CPU (fake_hip.cpp): how many iterations
a launch takes."""
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
