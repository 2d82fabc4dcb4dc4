"""Elements per workgroup of the operator launches against the number of
elements, where the measured choice changes (CPU: the launches are recorded by
fake_hip.cpp).  A workgroup holds its elements' (N+1)^2 columns in whole
wavefronts of 64."""
import pytest

import fakehip


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fakehip.build(tmp_path_factory.mktemp("fakehip"))


# order, mesh, use, elements per workgroup
CASES = [
    (2, (27, 27, 27), "plain", 7), (2, (36, 36, 37), "plain", 7), (2, (37, 37, 37), "plain", 3),
    (2, (40, 40, 40), "plain32", 7), (2, (43, 43, 43), "plain32", 3), (2, (27, 27, 27), "helm", 7),
    (3, (13, 13, 13), "plain", 4), (3, (35, 35, 35), "plain", 4), (3, (36, 36, 36), "plain", 16),
    (3, (29, 29, 30), "helm", 4), (3, (31, 31, 31), "helm", 16),
    (4, (20, 20, 20), "cg", 5), (4, (22, 22, 23), "cg", 15), (4, (25, 25, 25), "cg", 5), (4, (28, 28, 28), "cg", 15),
    (6, (16, 16, 16), "cg", 1), (6, (16, 16, 17), "cg", 9), (6, (17, 17, 17), "cg", 1),
    (6, (16, 16, 20), "plain32", 5), (6, (17, 17, 18), "plain32", 1),
    (7, (3, 3, 3), "cg", 4), (7, (4, 4, 4), "cg", 1),
    (8, (6, 6, 7), "plain", 1), (8, (7, 7, 7), "plain", 3), (8, (9, 9, 9), "plain", 3), (8, (8, 10, 10), "plain", 1),
    (8, (8, 8, 8), "helm", 1), (8, (9, 9, 9), "helm", 3), (8, (9, 9, 9), "plain32", 3),
    (11, (8, 8, 8), "helm", 1), (11, (9, 9, 9), "helm", 3), (11, (9, 9, 9), "plain", 3),
    (8, (9, 9, 9), "cg", 3), (11, (9, 9, 9), "cg", 3), (11, (8, 8, 8), "cg", 1), (11, (8, 10, 10), "cg", 1),
    (12, (9, 9, 9), "cg", 3), (10, (9, 9, 9), "cg", 1),
    (12, (9, 9, 9), "plain", 3), (12, (9, 9, 9), "helm", 1),
]


def test_elements_per_workgroup(runtime):
    fakehip.run(runtime, f"""
        for N, nel, use, epw in {CASES!r}:
            m, info = mesh(N, nel, fp32=use == "plain32")
            u, w = np.zeros(info.n_local), np.zeros(info.n_local)
            if use == "helm":
                L.check(lib.sem_set_helmholtz(m, u.ctypes.data, u.ctypes.data, None), "helmholtz")
            fake.fake_clear()
            if use == "cg":
                o = opts(fixed_iters=1, use_graph=0, profile=1)
                L.check(lib.sem_pcg_solve(m, u.ctypes.data, w.ctypes.data, C.byref(o), None, None), "solve")
            else:
                L.check(lib.sem_ax(m, 1 if use == "plain32" else 0, u.ctypes.data, w.ctypes.data, None, None), "ax")
            got = [fake.fake_block(i) for i in launches("ax_kernel")]
            want = -(-epw * (N + 1) ** 2 // 64) * 64
            assert got == [want], (N, nel, use, got, want)
            lib.sem_free(m)
        """)


def test_schwarz_assembly_lanes(runtime):
    """The sum of the local solves takes a lane per node while its columns
    leave the device idle, a lane per column beyond."""
    fakehip.run(runtime, """
        for N, nel, planes in ((7, (2, 2, 2), 8), (7, (8, 8, 13), 8), (7, (8, 8, 14), 1), (3, (8, 16, 16), 4),
                               (3, (8, 16, 17), 1), (12, (4, 4, 13), 13), (12, (4, 4, 14), 1)):
            m, info = mesh(N, nel)
            r, z = np.zeros(info.n_local), np.zeros(info.n_local)
            L.check(lib.sem_set_schwarz(m, 1, None), "schwarz")
            fake.fake_clear()
            L.check(lib.sem_precond_apply(m, r.ctypes.data, z.ctypes.data, None), "precond")
            (i,) = launches("assemble_kernel")
            per = max(1, 256 // (N + 1) ** 2)
            got = fake.fake_grid(i), fake.fake_grid_y(i)
            assert got == (-(-info.E // per), planes), (N, nel, got)
            lib.sem_free(m)
        """)
