"""The register engine of the ring stage at every transform length it takes in one launch (256 to 4096
points, whole rings and Bluestein convolutions, several rings to a workgroup): HEALPix sizes whose ring
counts leave workgroups partly filled and whose rings lie at both ends of each length, against the LDS
kernels in every ring mode and, where it is quick, against the oracle.

Tolerance against the LDS kernels: both compute each transform to a few eps log2 M, in different orders;
with M <= 4096 and the sums over rings that is below 1e-14 in FP64 (1e-12 asked) and 5e-7 in FP32 (2e-6
asked), as for the longer lengths."""
import numpy as np
import pytest

import akra_workloads as wl
from oracle.core import Oracle
from oracle.geometry import healpix_rings

from test_gpu_parity import check_alm, check_maps

pytestmark = pytest.mark.gpu

# (nside, lmax, nrhs): rings of 4 pixels only; whole rings below 256 points through Bluestein; belts of
# 256, 512, 1024 and 2048; caps that end just below and just past N = 2^k / 2; few and many orders per bin
SIZES = [(1, 2, 1), (2, 4, 2), (31, 40, 1), (32, 96, 3), (33, 20, 1), (64, 128, 1), (64, 256, 2), (65, 64, 1),
         (128, 256, 1), (129, 30, 4), (256, 300, 1), (257, 12, 2), (512, 64, 1), (520, 20, 1)]


def _plan(nside, lmax, prec, nrhs, engine):
    from paper_2606_06175_amd import Plan, akra
    akra.set_ring_register_engine(engine)
    try:
        print("plan nside=%d lmax=%d %s nrhs=%d engine=%d" % (nside, lmax, prec, nrhs, engine), flush=True)
        return Plan(nside, lmax, nrhs=nrhs, precision=prec, device="cuda:0")
    finally:
        akra.set_ring_register_engine(True)


def _rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / max(np.linalg.norm(np.ravel(b)), 1e-300))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nside,lmax,nrhs", SIZES)
def test_ring_lengths(nside, lmax, nrhs, prec):
    import torch
    dev = torch.device("cuda", 0)
    rings = healpix_rings(nside)
    npix = rings.npix
    sq = (lambda t: t[0].contiguous()) if nrhs == 1 else (lambda t: t)
    alm = [np.stack([wl.random_alm(lmax, 40 + 20 * c + k, lmin=0) for k in range(nrhs)]) for c in (0, 1)]
    hs = [np.stack(m) for m in zip(*[wl.random_maps(npix, 60 + k) for k in range(nrhs)])]
    g = np.random.default_rng(7)
    z = wl.pixel_vectors(nside)[2]
    masks = {"random": g.uniform(size=npix) < 0.7, "north": z > 0.2, "stripe": (z > -0.5) & (z < -0.4)}
    ninv = np.stack([g.uniform(5.0, 60.0, npix) for _ in range(nrhs)])
    A, h = [sq(torch.from_numpy(a).to(dev)) for a in alm], [sq(torch.from_numpy(a).to(dev)) for a in hs]
    w = sq(torch.from_numpy(ninv).to(dev))
    out = {}
    for engine in (True, False):
        p = _plan(nside, lmax, prec, nrhs, engine)
        res = [("synth", p.synth2(*A)), ("adjoint", p.adjoint2(*h))]
        for name, m in masks.items():
            res.append((name, p.apply_H(w, torch.from_numpy(m.astype(np.uint8)).to(dev), A[0], A[1], 0.01)))
        out[engine] = [(n, [t.cpu().numpy() for t in r]) for n, r in res]
        p.close()
    tol = 1e-12 if prec == "fp64" else 2e-6
    for (name, x), (_, y) in zip(out[True], out[False]):
        for u, v in zip(x, y):
            e = _rel(u, v)
            print("%s rel %.3e" % (name, e), flush=True)
            assert e < tol, (name, e)
    if (lmax + 1) * rings.nrings <= 20000 and nrhs == 1:
        o = Oracle(lmax, rings)
        t = 1e-12 if prec == "fp64" else 1e-5
        check_maps(*out[True][0][1], *o.synth(alm[0][0], alm[1][0]), rings, t)
        check_alm(np.stack(out[True][1][1]), np.stack(o.adjoint(hs[0][0], hs[1][0])), lmax, t)


@pytest.mark.parametrize("nside,lmax", [(8, 16), (64, 128), (100, 150)])
def test_ring_lengths_gradient(nside, lmax):
    # the gradient epilogue (ring mode 3); both solves stop at 1e-12, so 1e-9 as for the longer lengths
    import torch
    from paper_2606_06175_amd import AkraSolve
    dev = torch.device("cuda", 0)
    npix = 12 * nside * nside
    g = np.random.default_rng(8)
    mask = (g.uniform(size=npix) < 0.6).astype(np.uint8)
    ninv = g.uniform(5.0, 60.0, npix)
    maps = [m * mask for m in wl.random_maps(npix, 9)]
    cE = torch.from_numpy(wl.random_alm(lmax, 10)).to(dev)
    res = {}
    for engine in (True, False):
        p = _plan(nside, lmax, "fp64", 1, engine)
        t = [torch.tensor(v, dtype=torch.float64, device=dev, requires_grad=True) for v in (*maps, ninv)]
        xE, xB = AkraSolve.apply(t[0], t[1], t[2], torch.from_numpy(mask).to(dev), p, dict(tol=1e-12, maxiter=3000))
        L = (cE.real * xE.real + cE.imag * xE.imag).sum() + 0.5 * (xB.real ** 2 + xB.imag ** 2).sum()
        L.backward()
        res[engine] = [v.grad.cpu().numpy() for v in t]
        p.close()
    for x, y in zip(res[True], res[False]):
        assert _rel(x, y) < 1e-9
