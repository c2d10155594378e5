// Ring-stage helpers shared by the LDS kernels and the register engine (device code, gfx950): folding the
// orders of a ring into its bins and back.  Not part of the public ABI.
#pragma once
#include "akra_leg.h"

namespace akra {
// arguments of the ring kernels: MODE 0: F -> maps (o1, o2).  MODE 1: maps (g1, g2) x W -> G.  MODE 2: F ->
// maps x W -> G in place.  MODE 3 (gradient of the solve): F = Y K x as maps px; with o1, o2 holding
// q = Y K u, per pixel  o3 = M (omega q . (g - px) - c),   (o1, o2) = omega W q.
struct RingArgs {
    const double *g1, *g2;
    double *o1, *o2;
    const double *W;
    double *o3;
    const uint8_t *mask;
    const double *cdev;
};
// the rings of RS that run on the register engine (akra_ring16_f64.hip, akra_ring16_f32.hip)
template <typename T, int MODE>
void ring16_launch(Plan &P, const RingSet &RS, const RingArgs &a, int nrhs, bool split);

template <typename T> __device__ __forceinline__ cplx<T> to_t(double2 z) { return mk<T>((T)z.x, (T)z.y); }

// e^{i pi (k0 + k1 u) / den} for u = 0, 1, ... as a running FP64 product (one rounding per step)
struct PhaseSeq {
    double2 cur, step;
    __device__ __forceinline__ PhaseSeq(int64_t k0, int64_t k1, int64_t den)
        : cur(cis_pi<double>(k0, den)), step(cis_pi<double>(k1, den))
    {
    }
    __device__ __forceinline__ double2 next()
    {
        const double2 r = cur;
        cur = cmul<double>(cur, step);
        return r;
    }
};

// a / N for 0 <= a < 2^24 from a float reciprocal rN = 1 / N and one correction
__device__ __forceinline__ int udiv(int a, int N, float rN)
{
    int q = (int)((float)a * rN);
    const int r = a - q * N;
    if (r < 0) --q;
    else if (r >= N) ++q;
    return q;
}

// fold_bin / unfold_bin with the phase ph = e^{i pi bin / N} supplied (used when shift)
template <typename T>
__device__ __forceinline__ cplx<T> fold_bin_ph(const cplx<T> *__restrict__ F, int bin, int N, float rN, int shift,
                                               int lmax, const double2 &ph)
{
    const int tlo = -udiv(lmax + bin, N, rN);
    const int thi = (lmax >= bin) ? udiv(lmax - bin, N, rN) : -1;
    T sr = 0, si = 0;
    for (int t = tlo; t <= thi; ++t) {
        const int m = bin + N * t;
        cplx<T> f = (m >= 0) ? F[2 * m] : F[2 * (-m) + 1];
        if (shift && (t & 1)) f = mk<T>(-f.x, -f.y);
        sr += f.x;
        si += f.y;
    }
    cplx<T> s = mk<T>(sr, si);
    if (shift) s = cmul<T>(s, mk<T>((T)ph.x, (T)ph.y));
    return s;
}
template <typename T>
__device__ __forceinline__ void unfold_bin_ph(cplx<T> *__restrict__ G, int bin, int N, float rN, int shift, int lmax,
                                              cplx<T> y, const double2 &ph)
{
    if (shift) y = cmul<T>(y, mk<T>((T)ph.x, (T)-ph.y));
    const int tlo = -udiv(lmax + bin, N, rN);
    const int thi = (lmax >= bin) ? udiv(lmax - bin, N, rN) : -1;
    for (int t = tlo; t <= thi; ++t) {
        const int m = bin + N * t;
        const cplx<T> g = (shift && (t & 1)) ? mk<T>(-y.x, -y.y) : y;
        if (m > 0) G[2 * m] = g;
        else if (m < 0) G[2 * (-m) + 1] = g;
        else {
            G[0] = g;
            G[1] = g;
        }
    }
}

}  // namespace akra
