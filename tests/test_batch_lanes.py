"""Where the operators of a batch's orders are launched side by side in a
captured iteration, and where in turn (CPU: fake_hip.cpp records the streams)."""
import pytest

import fakehip


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    return fakehip.build(tmp_path_factory.mktemp("fakehip"))


# (order, elements) of the slots, lanes expected; precision
CASES = [
    ([(7, (4, 4, 4))], 1, 0),                                               # one order
    ([(5, (8, 8, 8)), (7, (8, 8, 8)), (5, (2, 2, 2))], 1, 0),               # two
    ([(2, (8, 8, 8)), (3, (8, 8, 8)), (4, (8, 8, 8))], 1, 0),               # short launches
    ([(2, (3, 3, 3)), (4, (3, 3, 3)), (6, (3, 3, 3)), (7, (3, 3, 3))], 1, 0),
    ([(5, (2, 2, 2)), (7, (2, 2, 2)), (9, (2, 2, 2))], 3, 0),
    ([(N, (2, 2, 2)) for N in range(2, 11)], 3, 0),
    ([(5, (6, 6, 6)), (7, (6, 6, 6)), (9, (6, 6, 6))], 1, 1),               # FP32 inner iterations
]


def test_lanes(runtime):
    fakehip.run(runtime, f"""
        for specs, lanes, precision in {CASES!r}:
            ms = [mesh(N, nel, fp32=True) for N, nel in specs]
            fake.fake_fill(1.0)  # right-hand sides of norm 1
            B = C.c_void_p()
            L.check(lib.sem_batch_create(16, 0, None, C.byref(B)), "create")
            fake.fake_fill(0.0)
            o, slot, keep = opts(precision=precision), C.c_int(), []
            for m, info in ms:
                b, x = np.ones(info.n_local), np.zeros(info.n_local)
                keep.append((b, x))
                L.check(lib.sem_batch_admit(B, m, b.ctypes.data, x.ctypes.data, C.byref(o), C.byref(slot), None), "admit")
            active = C.c_int()
            fake.fake_clear()
            L.check(lib.sem_batch_step(B, 1, 1, None, C.byref(active)), "step")
            ax = launches("batch_ax_kernelIfLi" if precision else "batch_ax_kernelIdLi")
            # the CG form (mode 2) of each order, once per captured iteration
            cg = [i for i in ax if b"ELi2E" in fake.fake_name(i)]
            assert len(cg) == len({{N for N, _ in specs}}), [fake.fake_name(i) for i in ax]
            assert len({{fake.fake_stream(i) for i in cg}}) == lanes, (specs, precision)
            lib.sem_batch_free(B)
            for m, _ in ms:
                lib.sem_free(m)
        """)
