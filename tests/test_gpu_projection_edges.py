"""Projection basis beyond one launch's vectors, and of any magnitude."""
import numpy as np
import pytest
import torch

import seeded_inputs as SI
from oracle.projection import ProjectionSpace
from test_gpu_projection import _box, _continuous, _dev, _host

pytestmark = pytest.mark.gpu


# eight vectors fill a launch: the counts around it, two and three launches
@pytest.mark.parametrize("count", [7, 8, 9, 16, 17, 25])
def test_many_vectors_against_the_oracle(semlib, oracle_mod, count):
    print(f"case: projection basis of {count}, box 3x3x2 N=4", flush=True)
    m, om = _box(semlib, oracle_mod, 4, (3, 3, 2), 5)
    P, ref = semlib.Projection(m, max_vectors=32), ProjectionSpace(om, 32)
    vs = [_continuous(om, 70 + s) for s in range(count)]
    for v in vs:
        assert P.add(_dev(v)) and ref.add(v)
    b = om.mass(SI.sin3_forcing(*om.coords()))
    xg, xo = _host(P.project(_dev(b))), ref.project(b)
    assert np.linalg.norm(xg - xo) <= 1e-11 * np.linalg.norm(xo)
    x = 0.5 * vs[0] - 2.0 * vs[-1]
    xb = _host(P.project(_dev(om.apply(x))))
    assert np.linalg.norm(xb - x) <= 1e-10 * np.linalg.norm(x)
    assert not P.add(_dev(vs[1] + vs[-1])) and len(P) == count
    P.close()
    m.close()


# a power of two on the solutions changes no bit of the guess; a vector with
# no norm is dropped and leaves the basis as it was
@pytest.mark.parametrize("power", [-450, -31, 450])
def test_magnitude_of_the_solutions(semlib, oracle_mod, power):
    print(f"case: projection of solutions times 2^{power}, box 3x2x2 N=5", flush=True)
    m, om = _box(semlib, oracle_mod, 5, (3, 2, 2), 3)
    P, Q = semlib.Projection(m, max_vectors=5), semlib.Projection(m, max_vectors=5)
    b = _dev(om.mass(SI.sin3_forcing(*om.coords())))
    for s in range(4):
        v = _continuous(om, 50 + s)
        assert P.add(_dev(v)) and Q.add(_dev(np.ldexp(v, power)))
    guess = P.project(b)
    assert torch.equal(guess, Q.project(b))
    for bad in (0.0, np.nan, np.inf):
        assert not Q.add(torch.full_like(b, bad)) and len(Q) == 4
    assert torch.equal(guess, Q.project(b))
    P.close()
    Q.close()
    m.close()
