"""Stages of a PCG iteration at sizes where latency is everything, against the two vector kernels of the same
iteration as the clock (best of many, so other work on the machine does not count).

Epilogue at Nside 128, lmax 256: its loads are on their way together.  One after the other it took 1.35 times the
vector kernels, together 0.98."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_epilogue_time():
    import torch
    from paper_2606_06175_amd import Plan
    nside, lmax = 128, 256
    npix = 12 * nside * nside
    dev = torch.device("cuda", 0)
    g = np.random.default_rng(1)
    mask = torch.from_numpy((np.arange(npix) % 3 > 0).astype(np.uint8)).to(dev)
    g1, g2 = (torch.from_numpy(g.normal(size=npix)).to(dev) for _ in "12")
    ninv = torch.from_numpy(g.uniform(5.0, 60.0, npix)).to(dev)
    p = Plan(nside, lmax, precision="fp64", device=dev)
    p.set_timing(True)
    best = {}
    for rep in range(60):
        p.cg_start(g1, g2, ninv, mask)
        p.stage_times()
        p.cg_step(10)
        for stage, (ms, n) in p.stage_times().items():
            best[stage] = min(best.get(stage, 1e9), 1e3 * ms / n)
    p.close()
    print({k: round(v, 2) for k, v in best.items()}, flush=True)
    assert best["epilogue"] <= 1.2 * best["cg_vec"]


def test_classes_of_a_small_plan():
    """Group classes too short to pay for a second stream: an apply of two classes against one of all rings in one
    class (Nside 48, lmax 48: 85 us on two streams, 75 on one, all rings 66)."""
    import time

    import torch
    import akra_workloads as wl
    from paper_2606_06175_amd import Plan
    nside, lmax = 48, 48
    npix = 12 * nside * nside
    dev = torch.device("cuda", 0)
    g = np.random.default_rng(1)
    z = wl.pixel_vectors(nside)[2]
    mask = torch.from_numpy(((z < 0.1) & (z > -0.9)).astype(np.uint8)).to(dev)
    ninv = torch.from_numpy(g.uniform(5.0, 60.0, npix)).to(dev)
    a = [torch.from_numpy(wl.random_alm(lmax, k)).to(dev) for k in (1, 2)]
    plans = {}
    for skip in (True, False):
        plans[skip] = Plan(nside, lmax, precision="fp64", device=dev)
        plans[skip].set_skip_unweighted(skip)
    best = {True: 1e9, False: 1e9}
    for rep in range(100):
        for skip, p in plans.items():
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                p.apply_H(ninv, mask, *a, 0.02)
            torch.cuda.synchronize()
            if rep >= 10:
                best[skip] = min(best[skip], (time.perf_counter() - t0) / 5)
    w = plans[True].work_weighted()
    for p in plans.values():
        p.close()
    print("apply: skipping %.1f us, all rings %.1f us" % (1e6 * best[True], 1e6 * best[False]), flush=True)
    assert w["synth_two"] > 0 and w["synth_one"] > 0
    assert best[True] <= 1.25 * best[False]
