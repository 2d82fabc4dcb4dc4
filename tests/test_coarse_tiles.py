"""The lists of the coarse term's tiles (CPU): against a walk over the rows of
A0 (coarse_tiles_check.cpp), and that setting the coarse term up sends none of
them -- they are written on the device from the lattice."""
import os
import subprocess

import fakehip

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lists_are_those_of_the_rows(tmp_path):
    from paper_2109_03592_amd import build as B
    exe = tmp_path / "coarse_tiles_check"
    src = os.path.join(ROOT, "tests", "coarse_tiles_check.cpp")
    subprocess.run([B.HIPCC, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", src, "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout + r.stderr


def test_set_up_sends_the_rows_alone(tmp_path):
    """Per element its 64 block entries and 8 corners, per vertex its row and
    its inverse diagonal, and the order's small tables."""
    fakehip.run(fakehip.build(tmp_path), """
        for nel, k in (((6, 5, 4), 4), ((16, 16, 16), 4), ((24, 24, 20), 9)):
            m, info = mesh(2, nel)
            nvert = (nel[0] + 1) * (nel[1] + 1) * (nel[2] + 1)
            fake.fake_fill(1.0)  # a positive coarse operator
            before = fake.fake_copied()
            L.check(lib.sem_set_coarse(m, k, 0.1, None), "coarse")
            fake.fake_fill(0.0)
            sent = fake.fake_copied() - before
            assert sent <= 8 * 64 * info.E + 4 * 8 * info.E + 8 * 33 * nvert + 1024, (nel, sent)
            lib.sem_free(m)
        """)
