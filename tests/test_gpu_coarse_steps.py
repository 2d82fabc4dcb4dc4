"""The coarse term's Chebyshev solve over its ranges: step counts around what
one launch takes, vertex lattices from less than one tile to more tiles of the
largest size than workgroups, periodic wraps inside a tile's surroundings."""
import numpy as np
import pytest
import torch

import seeded_inputs as SI
from oracle.coarse import CoarseOracle

pytestmark = pytest.mark.gpu


# no product with A0, one, the three of a launch, two launches, three; periodic
# lattices narrower than a tile's surroundings; one tile
@pytest.mark.parametrize("N,nel,periodic,k", [(3, (4, 3, 5), (0, 1, 0), k) for k in (1, 2, 3, 4, 5, 6, 9)] +
                         [(3, (2, 2, 3), (1, 1, 0), 4), (4, (2, 1, 1), (0, 0, 0), 5), (2, (2, 7, 9), (1, 0, 1), 4)])
def test_chebyshev_solve(semlib, oracle_mod, N, nel, periodic, k):
    print(f"case: coarse steps N={N} nel={nel} periodic={periodic} k={k}", flush=True)
    m = semlib.box_mesh(N, nel, periodic=periodic)
    om = oracle_mod.OracleMesh(N, nel, periodic=periodic)
    r = SI.uniform_global_values(om.nglob, seed=40 + k)[om.numbering()] * (om.local_mask() == 0)
    C = CoarseOracle(om, k=k, frac=0.05)
    ref = C.inv * r + C.coarse(r)
    m.set_coarse(k, 0.05)
    z = m.precond(torch.from_numpy(np.ascontiguousarray(r)).cuda()).cpu().numpy()
    assert np.linalg.norm(z - ref) <= 1e-12 * np.linalg.norm(ref)
    assert np.max(np.abs(z - ref)) <= 1e-12 * np.max(np.abs(ref))
    m.close()


def _unit_cubes(semlib, nel):
    g = [np.arange(n + 1, dtype=np.float64) for n in nel]
    z, y, x = np.meshgrid(g[2], g[1], g[0], indexing="ij")
    return semlib.box_mesh(1, nel, vertices=np.stack([x, y, z], axis=-1).reshape(-1, 3), periodic=(1, 1, 1))


# unit cubes, periodic in all directions: on a larger box of whole periods the
# result repeats that of one period.  Tile edges 4, 6 and 8, the last with more
# tiles than workgroups (1080 of 1024)
@pytest.mark.parametrize("nel", [(24, 16, 24), (32, 40, 32), (96, 80, 72)])
@pytest.mark.parametrize("k", [4, 6])
def test_larger_lattices_repeat_a_period(semlib, nel, k):
    print(f"case: coarse tiles nel={nel} k={k}", flush=True)
    s, m = _unit_cubes(semlib, (8, 8, 8)), _unit_cubes(semlib, nel)
    vals = torch.from_numpy(SI.uniform_global_values(s.n_global, seed=k)).cuda()
    r = s.scatter(vals)
    e = torch.arange(m.n_local // 8, device="cuda")
    ex, ey, ez = e % nel[0], e // nel[0] % nel[1], e // (nel[0] * nel[1])
    period = ex % 8 + 8 * (ey % 8 + 8 * (ez % 8))
    for q in (s, m):
        q.set_coarse(k, 0.05)
    ref = s.precond(r).view(-1, 8)[period].reshape(-1)
    z = m.precond(r.view(-1, 8)[period].reshape(-1).contiguous())
    assert (z - ref).abs().max() <= 1e-13 * ref.abs().max()
    s.close()
    m.close()


# slots whose chains take one, two and three launches share a batch: each is
# the solve alone in a batch, and the residual reaches the tolerance
def test_batched_chains_of_different_lengths(semlib):
    print("case: batched coarse chains k=1,4,6,9", flush=True)
    meshes, bs = [], []
    for k, (N, nel) in zip((1, 4, 6, 9), ((5, (4, 4, 3)), (7, (3, 4, 4)), (4, (6, 5, 4)), (9, (3, 3, 2)))):
        m = semlib.box_mesh(N, nel, vertices=SI.jittered_box_vertices(nel, seed=k), with_fp32=True)
        m.set_coarse(k, 0.05)
        meshes.append(m)
        bs.append(m.scatter(torch.from_numpy(SI.uniform_global_values(m.n_global, k)).cuda()))
    for precision in ("fp64", "mixed"):
        B = semlib.Batch(max_slots=4)
        xs, res = B.solve(meshes, bs, tol=1e-10, precision=precision)
        for m, b, x, r in zip(meshes, bs, xs, res):
            (alone,), (ra,) = B.solve([m], [b], tol=1e-10, precision=precision)
            assert r.ok and ra.ok and r.iterations == ra.iterations and torch.equal(x, alone)
        B.close()
    for m in meshes:
        m.close()
