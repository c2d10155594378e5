"""Low degrees on many rings (GPU): the scalar form divides by sin^2(theta), which shows in the rounding where the
recurrence runs over few oscillations, so the groups within 40 / lmax of a pole keep the spin form.

Synthesis error of the spin form by itself (against 64 bits more): 1.9e-15 of the ring's rms at 0.15 rad and 1.0e-15 at
0.2 for lmax 16, 3.2e-15 for lmax 64; the ring stage adds about eps log2 M = 1e-15.  Twice the sum, 6e-15 and 8e-15,
is allowed for the rms over the rings of a group; the scalar form has 2e-14 and 6e-15 of its own at the first of them.
The plans on both sides of the rule: 1e-12, as for all forms."""
import numpy as np
import pytest

import akra_workloads as wl
from oracle.core import Oracle
from oracle.geometry import healpix_rings

from test_gpu_parity import check_alm, check_maps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nside,lmax,tol", [(350, 16, 6e-15), (350, 64, 8e-15), (5, 4, 6e-15)])
def test_low_degree_rounding(nside, lmax, tol):
    import torch
    from paper_2606_06175_amd import Plan
    rings = healpix_rings(nside)
    a = [wl.random_alm(lmax, s) for s in (1, 2)]
    ref = Oracle(lmax, rings).synth(*a)
    p = Plan(nside, lmax, device="cuda:0")
    got = [v.cpu().numpy() for v in p.synth2(*(torch.from_numpy(v).to("cuda:0") for v in a))]
    p.close()
    e2 = (got[0] - ref[0]) ** 2 + (got[1] - ref[1]) ** 2
    r2 = ref[0] ** 2 + ref[1] ** 2
    first = 64 if nside > 64 else 0
    err = []
    for r in range(first, first + min(16, rings.nrings)):
        s = slice(int(rings.ofs[r]), int(rings.ofs[r]) + int(rings.nphi[r]))
        err.append(np.sqrt(e2[s].sum() / r2[s].sum()))
    rms = float(np.sqrt(np.mean(np.square(err))))
    print("nside %d lmax %d: error %.2e of the ring's rms" % (nside, lmax, rms), flush=True)
    assert rms < tol


@pytest.mark.parametrize("prec,tol,nrhs", [("fp64", 1e-12, 1), ("fp32", 1e-5, 1), ("fp32", 1e-5, 3)])
@pytest.mark.parametrize("nside,lmax", [(65, 47), (65, 48), (260, 95), (260, 99), (3, 12)])
def test_both_sides(nside, lmax, prec, tol, nrhs):
    # the second group begins 0.839 rad (Nside 65) and 0.204, the third 0.406 rad (Nside 260) from the pole
    import torch
    from paper_2606_06175_amd import Plan
    rings = healpix_rings(nside)
    o = Oracle(lmax, rings)
    a = [wl.random_alm(lmax, s) for s in (1, 2)]
    h = wl.random_maps(rings.npix, 3)
    rep = (lambda v: torch.from_numpy(v).to("cuda:0")) if nrhs == 1 else \
        (lambda v: torch.from_numpy(np.stack([v] * nrhs)).to("cuda:0"))
    p = Plan(nside, lmax, nrhs=nrhs, precision=prec, device="cuda:0")
    last = lambda v: v.cpu().numpy().reshape(nrhs, -1)[-1]
    g = [last(v) for v in p.synth2(*(rep(v) for v in a))]
    check_maps(g[0], g[1], *o.synth(*a), rings, tol)
    got = np.stack([last(v) for v in p.adjoint2(*(rep(v) for v in h))])
    p.close()
    check_alm(got, np.stack(o.adjoint(*h)), lmax, tol)
