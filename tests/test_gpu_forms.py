"""The two forms of the Legendre kernels (GPU): 64-pair groups that begin near a pole run the spin-weighted
recurrences, the others scalar functions to degree lmax + 2 through a five-point stencil.  Sizes where a
group boundary, the first and last degrees, or the last pairs of a group fall at an edge, against the
oracle per ring and per m.

Tolerance: FP64 1e-12.  The recurrence's phase error is about sqrt(l) eps / theta, with l <= 130 and the
nearest ring of a scalar group at 0.2 rad: 1e-14; the polar rings' (0.003 rad at the smallest, lmax 12)
about 3e-13.  FP32 plans store F and G as floats and run FP32 FFTs: 1e-5, as
elsewhere."""
import numpy as np
import pytest

import akra_workloads as wl
from oracle.core import Oracle
from oracle.geometry import healpix_rings

from test_gpu_parity import check_alm, check_maps

pytestmark = pytest.mark.gpu

# (nside, lmax): one pair past the first group; lmax 2 and 3 (every degree within the stencil's reach of
# both ends); lmax + 2 just below, at and past a multiple of the eight-degree chunk; many empty groups
SIZES = [(33, 2), (33, 3), (33, 130), (64, 5), (65, 6), (70, 9), (128, 17), (260, 12)]


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("nside,lmax", SIZES)
def test_forms_match_oracle(nside, lmax, prec, tol):
    import torch
    from paper_2606_06175_amd import Plan
    print("nside %d lmax %d %s" % (nside, lmax, prec), flush=True)
    dev = torch.device("cuda", 0)
    rings = healpix_rings(nside)
    o = Oracle(lmax, rings)
    a = [wl.random_alm(lmax, s, lmin=0) for s in (1, 2)]
    h = wl.random_maps(rings.npix, 3)
    ta, th = [torch.from_numpy(v).to(dev) for v in a], [torch.from_numpy(v).to(dev) for v in h]
    p = Plan(nside, lmax, precision=prec, device=dev)
    g = [v.cpu().numpy() for v in p.synth2(*ta)]
    check_maps(g[0], g[1], *o.synth(*a), rings, tol)
    got = np.stack([v.cpu().numpy() for v in p.adjoint2(*th)])
    check_alm(got, np.stack(o.adjoint(*h)), lmax, tol)
    # weight on the north half, the south half, and a polar cap with a stripe on the other side
    z = wl.pixel_vectors(nside)[2]
    ninv = np.random.default_rng(4).uniform(5.0, 60.0, rings.npix)
    for name, foot in (("north", z > 0.1), ("south", z < -0.1), ("mixed", (z > 0.995) | ((z < -0.2) & (z > -0.5)))):
        print(name, flush=True)
        mask = foot.astype(np.uint8)
        y = p.apply_H(torch.from_numpy(ninv).to(dev), torch.from_numpy(mask).to(dev), ta[0], ta[1], 0.02)
        ref = o.apply_H(np.stack(a), o.weights(ninv, mask), 0.02)
        check_alm(np.stack([v.cpu().numpy() for v in y]), ref, lmax, tol)
    p.close()


# (nside, lmax, nrhs): groups of at most four right-hand sides (16-column products) and of eight (32
# columns), full and padded, alone and one after the other; degrees just past a round (4 or 8) and past a
# 64-degree chunk; one group, spin and scalar groups, many groups that never enter
BATCHED = [(33, 2, 2), (33, 66, 4), (64, 61, 5), (70, 9, 8), (100, 130, 12), (128, 63, 3), (260, 12, 13)]


@pytest.mark.parametrize("nside,lmax,nrhs", BATCHED)
def test_batched_forms_match_oracle(nside, lmax, nrhs):
    # FP32 products and sums of FP64 recurrence values: each coefficient and value is rounded once (6e-8),
    # the division by sin^2 amplifies that by at most 11 (0.3 rad), so 1e-5 holds with room, per ring and
    # per m; the spin groups within 0.3 rad keep the 1e-5 of the FP32 difference form
    import torch
    from paper_2606_06175_amd import Plan
    print("nside %d lmax %d nrhs %d" % (nside, lmax, nrhs), flush=True)
    dev = torch.device("cuda", 0)
    rings = healpix_rings(nside)
    o = Oracle(lmax, rings)
    A, B = (np.stack([wl.random_alm(lmax, 10 * s + k, lmin=0) for k in range(nrhs)]) for s in (3, 9))
    z = wl.pixel_vectors(nside)[2]
    mask = ((z < 0.6) & (z > -0.9)).astype(np.uint8)
    ninv = np.stack([np.random.default_rng(40 + k).uniform(5.0, 60.0, rings.npix) for k in range(nrhs)])
    p = Plan(nside, lmax, nrhs=nrhs, precision="fp32", device=dev)
    tA, tB = torch.from_numpy(A).to(dev), torch.from_numpy(B).to(dev)
    g1, g2 = (v.cpu().numpy() for v in p.synth2(tA, tB))
    yE, yB = (v.cpu().numpy() for v in p.apply_H(torch.from_numpy(ninv).to(dev), torch.from_numpy(mask).to(dev), tA,
                                                 tB, 0.02))
    for k in sorted({0, nrhs // 2, nrhs - 1}):
        check_maps(g1[k], g2[k], *o.synth(A[k], B[k]), rings, 1e-5)
        ref = o.apply_H(np.stack([A[k], B[k]]), o.weights(ninv[k], mask), 0.02)
        check_alm(np.stack([yE[k], yB[k]]), ref, lmax, 1e-5)
    p.close()


@pytest.mark.parametrize("prec,nrhs", [("fp64", 1), ("fp32", 1), ("fp32", 3)])
def test_degrees_below_two_take_no_part(prec, nrhs):
    # spin-2 transforms start at l = 2: whatever l = 0 and 1 hold, also NaN or infinity, changes nothing
    import torch
    from paper_2606_06175_amd import Plan
    nside, lmax = 33, 20
    dev = torch.device("cuda", 0)
    low = [0, 1, lmax + 1]  # (l, m) = (0, 0), (1, 0), (1, 1)
    p = Plan(nside, lmax, nrhs=nrhs, precision=prec, device=dev)
    x = np.stack([[wl.random_alm(lmax, 5 * c + k, lmin=0) for k in range(nrhs)] for c in (0, 1)])
    out = []
    for bad in (0.0, np.nan, np.inf):
        y = x.copy()
        y[..., low] = bad
        t = [torch.from_numpy(v[0] if nrhs == 1 else v).to(dev).contiguous() for v in y]
        out.append([v.cpu().numpy() for v in p.synth2(*t)])
    p.close()
    for o in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(o, out[0]))
