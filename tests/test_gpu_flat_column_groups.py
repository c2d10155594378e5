"""Grids on both sides of the flat-sky column pass's choice between one and four columns per workgroup (512 columns
below 1024 points, 1024 from there on), against the flat oracle.  Tolerance 1e-12: FP64 transforms of at most 2^22
points, a few eps log2 n."""
import numpy as np
import pytest

from oracle.flat import FlatOracle

from test_gpu_flat import TOL, _c, _plan, _rand, _t, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(512, 256), (512, 1024), (1024, 256), (1024, 1024), (2048, 1024), (4096, 1024)])
def test_column_groups(nx, ny):
    o = FlatOracle(nx, ny)
    p = _plan(nx, ny)
    a, b = _rand(ny, nx, nx + ny)
    g = np.random.default_rng(nx)
    ninv, mask = g.uniform(1.0, 9.0, (ny, nx)), (g.uniform(size=(ny, nx)) < 0.6).astype(np.uint8)
    lam = o.lambda_eff(ninv, mask)
    W = o.weights(ninv, mask)
    z = a + 1j * b
    assert rel(_c(p, *p.synth(_t(a), _t(b))), o.synth(z)) < TOL
    assert rel(_c(p, *p.apply_H(_t(ninv), _t(mask), _t(a), _t(b), lam)), o.apply_H(z, W, lam)) < TOL
    assert rel(_c(p, *p.rhs(_t(a), _t(b), _t(ninv), _t(mask))), o.rhs(a, b, W)) < TOL
