"""Ring stage of small plans: too few rings to fill the device with several rings per workgroup, so their short
transforms run on the LDS kernels, both kinds in one launch.

The plans on both sides of that rule are compared with plans whose register engine is off: both compute each
transform to a few eps log2 M in different orders, so 1e-12 in FP64 and 2e-6 in FP32 (as for the ring lengths)."""
import numpy as np
import pytest

import akra_workloads as wl

pytestmark = pytest.mark.gpu


def _plan(nside, lmax, prec, nrhs, engine):
    from paper_2606_06175_amd import Plan, akra
    akra.set_ring_register_engine(engine)
    try:
        print("plan nside=%d lmax=%d %s nrhs=%d engine=%d" % (nside, lmax, prec, nrhs, engine), flush=True)
        return Plan(nside, lmax, nrhs=nrhs, precision=prec, device="cuda:0")
    finally:
        akra.set_ring_register_engine(True)


def _operands(nside, lmax, nrhs, full):
    import torch
    dev = torch.device("cuda", 0)
    npix = 12 * nside * nside
    g = np.random.default_rng(3)
    sq = (lambda t: t[0].contiguous()) if nrhs == 1 else (lambda t: t)
    alm = [sq(torch.from_numpy(np.stack([wl.random_alm(lmax, 9 + 40 * c + k) for k in range(nrhs)])).to(dev)) for c in (0, 1)]
    ninv = sq(torch.from_numpy(g.uniform(5.0, 60.0, (nrhs, npix))).to(dev))
    mask = np.ones(npix, bool) if full else g.uniform(size=npix) < 0.5
    return alm, ninv, torch.from_numpy(mask.astype(np.uint8)).to(dev)


# rings x right-hand sides on both sides of 640: 612, 663, 630, 693, 635, 643; and FP64 plans whose transforms lie above
# (762, 765 and 765) and whose applies, one right-hand side at a time, below
@pytest.mark.parametrize("nside,lmax,prec,nrhs", [(13, 20, "fp32", 12), (13, 20, "fp32", 13), (16, 60, "fp32", 10),
                                                  (16, 24, "fp32", 11), (159, 40, "fp64", 1), (161, 40, "fp64", 1),
                                                  (161, 200, "fp32", 1), (32, 64, "fp64", 6),
                                                  (64, 128, "fp64", 3), (64, 250, "fp64", 3)])
def test_both_sides(nside, lmax, prec, nrhs):
    alm, ninv, mask = _operands(nside, lmax, nrhs, False)
    out = []
    for engine in (True, False):
        p = _plan(nside, lmax, prec, nrhs, engine)
        maps = p.synth2(*alm)
        out.append([x.cpu().numpy() for x in (*maps, *p.adjoint2(*maps), *p.apply_H(ninv, mask, *alm, 0.02))])
        p.close()
    for a, b in zip(*out):
        assert np.linalg.norm(a - b) <= (1e-12 if prec == "fp64" else 2e-6) * np.linalg.norm(b)


@pytest.mark.parametrize("nside,lmax", [(16, 16), (32, 80), (45, 112)])
def test_ring_stage_time(nside, lmax):
    """The default is no slower than the LDS kernels alone (Nside 32: 13 us; several rings per workgroup take 20)."""
    alm, ninv, mask = _operands(nside, lmax, 1, True)
    plans = {e: _plan(nside, lmax, "fp64", 1, e) for e in (True, False)}
    best = {}
    for p in plans.values():
        p.set_timing(True)
    for rep in range(60):
        for e, p in plans.items():
            p.apply_H(ninv, mask, *alm, 0.02)
            ms, n = p.stage_times()["ring"]
            if rep >= 10:
                best[e] = min(best.get(e, 1e9), ms / n)
    for p in plans.values():
        p.close()
    print("ring stage: default %.1f us, LDS kernels %.1f us" % (1e3 * best[True], 1e3 * best[False]), flush=True)
    assert best[True] <= 1.25 * best[False]
