"""The operator's elements per workgroup are chosen by order, precision, use
and element count; the results do not depend on the choice."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# either side of 1024 elements (one element per workgroup from order 8 on), the
# orders whose counts differ between the plain and Helmholtz launches, and
# ragged last tiles
@pytest.mark.parametrize("N,nel", [(2, (5, 4, 3)), (3, (5, 5, 7)), (4, (7, 3, 3)), (6, (3, 3, 4)), (9, (8, 8, 16)),
                                   (9, (8, 8, 17)), (11, (11, 11, 9)), (12, (2, 3, 2)), (12, (11, 10, 10))])
@pytest.mark.parametrize("helm", [False, True])
def test_default_tile_gives_the_bits_of_any_other(semlib, N, nel, helm):
    print(f"case: tile choice N={N} nel={nel} helm={helm}", flush=True)
    m = semlib.box_mesh(N, nel, with_fp32=True)
    g = torch.Generator().manual_seed(3)
    u, h1, h2 = (0.5 + torch.rand(m.n_local, generator=g, dtype=torch.float64).cuda() for _ in range(3))
    if helm:
        m.set_helmholtz(h1, h2)
    fields = [u, u.to(torch.float32)]
    ref = [m.ax(v) for v in fields]
    for epw in (1, 2):
        m.set_operator_config(epw, 0)
        for v, w in zip(fields, ref):
            assert torch.equal(w, m.ax(v)), (v.dtype, epw)
    m.close()
