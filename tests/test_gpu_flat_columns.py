"""The flat-sky column pass (one or, from 512 columns on, four columns of 256 to 4096 points per workgroup) at
every length it takes, with the fewest columns and more, and the lengths on either side that keep the transposed row pass, against
the flat oracle: synthesis, adjoint, operator and right-hand side.

Tolerance 1e-12: FP64 transforms of at most 2^21 points, a few eps log2 n."""
import numpy as np
import pytest

from oracle.flat import FlatOracle

from test_gpu_flat import TOL, _c, _plan, _rand, _t, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(128, 16), (256, 4), (256, 32), (512, 8), (1024, 4), (1024, 64), (2048, 16),
                                   (4096, 4), (4096, 32), (8192, 8), (256, 256), (256, 512), (512, 512),
                                   (1024, 512), (2048, 512), (4096, 512)])
def test_columns_match_oracle(nx, ny):
    o = FlatOracle(nx, ny)
    p = _plan(nx, ny)
    a, b = _rand(ny, nx, nx + ny)
    g = np.random.default_rng(nx)
    ninv, mask = g.uniform(1.0, 9.0, (ny, nx)), (g.uniform(size=(ny, nx)) < 0.6).astype(np.uint8)
    lam = o.lambda_eff(ninv, mask)
    W = o.weights(ninv, mask)
    z = a + 1j * b
    assert rel(_c(p, *p.synth(_t(a), _t(b))), o.synth(z)) < TOL
    assert rel(_c(p, *p.adjoint(_t(a), _t(b))), o.adjoint(z)) < TOL
    assert rel(_c(p, *p.apply_H(_t(ninv), _t(mask), _t(a), _t(b), lam)), o.apply_H(z, W, lam)) < TOL
    assert rel(_c(p, *p.rhs(_t(a), _t(b), _t(ninv), _t(mask))), o.rhs(a, b, W)) < TOL
