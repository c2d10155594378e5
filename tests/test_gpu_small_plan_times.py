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
