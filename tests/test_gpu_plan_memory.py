"""Device memory of plans: what a right-hand side of a batched plan costs, and tables that only FP32 plans hold."""
import pytest

pytestmark = pytest.mark.gpu


def _bytes(nside, lmax, prec, nrhs):
    from paper_2606_06175_amd import Plan
    p = Plan(nside, lmax, nrhs=nrhs, precision=prec, device="cuda:0")
    b = p.device_bytes
    p.close()
    return b


@pytest.mark.parametrize("nside,lmax", [(32, 64), (64, 128), (200, 300)])
def test_right_hand_side_of_a_batch(nside, lmax):
    # F and G, weights, the six solver vectors, 40 KB of partial sums; no records of the single-vector transforms
    nalm, nrings, npix = (lmax + 1) * (lmax + 2) // 2, 4 * nside - 1, 12 * nside * nside
    per = (_bytes(nside, lmax, "fp32", 16) - _bytes(nside, lmax, "fp32", 9)) / 7
    need = 32 * nrings * (lmax + 1) + 8 * npix + 6 * 32 * nalm
    print("per right-hand side %.0f bytes, buffers %.0f" % (per, need), flush=True)
    assert per <= need + 40000


@pytest.mark.parametrize("nside,lmax", [(65, 130), (200, 300)])
def test_fp64_plans_hold_no_fp32_spectra(nside, lmax):
    """Chirp spectra of the Bluestein rings in FP32 (a complex float per point of each distinct convolution) are an
    FP32 plan's; the synthesis records take 40 and 48 bytes, the tables of the recurrences 60 + 64 per (l, m)."""
    b64, b32 = _bytes(nside, lmax, "fp64", 1), _bytes(nside, lmax, "fp32", 1)
    print("fp64 %d fp32 %d" % (b64, b32), flush=True)
    lengths = [n for n in {4 * min(i, nside) for i in range(1, nside + 1)} if n & (n - 1)]
    assert b32 - b64 >= sum(8 * (2 * n - 1) for n in lengths)
