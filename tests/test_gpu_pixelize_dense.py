"""Pixel buckets with many galaxies for each of few pixels, which are sorted by pixel in LDS: the smallest such
buckets, batches (512 galaxies) filled to the edge, pixels that take a whole batch, and buckets of both kinds in
one workgroup, against the oracle bit for bit; and the time of a crowded bucket."""
import numpy as np
import pytest

import akra_workloads as wl
from oracle.pixelize import pixelize

pytestmark = pytest.mark.gpu


def _patch(n, pixels, nside, seed):
    """n galaxies over some consecutive pixels of the ring past the equator."""
    g = np.random.default_rng(seed)
    c = wl.make_catalog(n, 3)
    c["z"] = np.full(n, -2.0 / (3 * nside))
    c["phi"] = (g.integers(0, pixels, n) + 0.75) * (2 * np.pi / (4 * nside))
    return c


def _compare(nside, c):
    import torch
    from paper_2606_06175_amd import Plan
    print("nside %d galaxies %d" % (nside, len(c["z"])), flush=True)
    args = [c[k] for k in ("z", "phi", "e1", "e2", "w")]
    ref = pixelize(nside, *args, 0.7, 0.26, 1.5)
    p = Plan(nside, 2, device="cuda:0")
    o = p.pixelize(*(torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in args), 0.7, 0.26, 1.5)
    p.close()
    for k in ("g1", "g2", "ninv", "neff", "mask"):
        assert np.array_equal(o[k].cpu().numpy(), ref[k]), k


# 16, 32 and 64 pixels a bucket (128 at Nside 148); at 16 the dense buckets begin with 65 galaxies
@pytest.mark.parametrize("nside,pixels,n", [(64, 16, 64), (64, 16, 65), (64, 16, 511), (64, 16, 512), (64, 16, 513),
                                            (64, 1, 1537), (74, 32, 129), (74, 100, 5000), (104, 70, 4097),
                                            (105, 200, 20000), (128, 64, 257), (147, 3, 30000), (148, 300, 30000)])
def test_dense_bit_exact(nside, pixels, n):
    a, b = _patch(n, pixels, nside, n), wl.make_catalog(3000, 5)
    c = {k: np.concatenate([a[k], b[k]]) for k in ("z", "phi", "e1", "e2", "w")}
    order = np.random.default_rng(2).permutation(len(c["z"]))
    c = {k: v[order] for k, v in c.items()}
    c["w"][::31] = 0.0
    _compare(nside, c)


def test_crowded_bucket_time():
    """1e6 galaxies on 16 pixels of Nside 64, one bucket: 38 ms with one galaxy per pixel and turn, 12 ms sorted."""
    import time

    import torch
    from paper_2606_06175_amd import Plan
    c = _patch(1000000, 16, 64, 1)
    p = Plan(64, 2, device="cuda:0")
    a = [torch.from_numpy(np.ascontiguousarray(c[k])).to("cuda:0") for k in ("z", "phi", "e1", "e2", "w")]
    best = 1e9
    for _ in range(4):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        p.pixelize(*a, 0.7, 0.26, 1.5)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    p.close()
    print("crowded bucket: %.2f ms" % (1e3 * best), flush=True)
    assert best < 0.015
