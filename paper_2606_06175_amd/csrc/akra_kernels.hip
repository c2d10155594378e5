// Device kernels of libakra for CDNA4 (gfx950).
//
// Operator chain of the matrix-free H v (paper Sec. II.B, storage problem):
//   prologue      x -> K_l x                                   (harmonic diagonal, eq. Dl_kernel)
//   leg_synth     alm -> F_r(+-m) per ring                      (inverse SHT, Legendre stage)
//   ring          F -> fold -> inverse DFT -> x W -> DFT -> unfold -> G     (SHT ring stage + N^-1 M)
//   leg_adj       G -> partial sums of 2h_lm, -2h_lm            (adjoint SHT, Legendre stage)
//   epilogue      E/B combination (eq. EB_decomp), K_l, + lambda_eff x   (eq. ML_estimator_reg)
#include <type_traits>

#include "akra_ring.h"

namespace akra {

// ------------------------------------------------------------------------------------------------
// Entry states (plan build).  One wave per (m, 64-pair group) runs the FP64 recurrence from the
// seeds at l0 (max(m, 2) for the first nspin groups, which run the spin form, m for the others) with
// the rescaling of the Legendre kernels' ramp (two steps, then a rescale), and stops at the first
// degree where some pair of the group contributes: it has left the scaled range and reaches the form's
// bound.  FP64 plans take 2^-100 (spin) and 2^-105 (scalar, whose sums are divided by sin^2 theta): the
// values are of order one where they oscillate, so the terms of a group that is still below that
// everywhere change a sum by far less than FP64 rounding (2^-53), and skipping them saves about 5% of
// the triples at lmax 4096.  FP32 plans take 2^-44 and 2^-49.  The state at the last degree l0 + 8q
// before it is stored with that degree; a group that never contributes up to its last degree is
// marked ENT_SKIP.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_entry(const double *__restrict__ seed2, const double *__restrict__ seedm2,
                                               const int *__restrict__ seedk, const double *__restrict__ pair_z,
                                               const Coef64 *__restrict__ coef, const double *__restrict__ sa,
                                               Ent64 *__restrict__ ent, int *__restrict__ entk,
                                               int *__restrict__ entl, int lmax, int npairs, int ng, int gpb,
                                               int nspin, double live_spin, double live_scalar)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int m = blockIdx.x / gpb;
    const int g = (blockIdx.x - m * gpb) * 4 + wave;
    if (m > lmax || g >= ng) return;
    const int p = g * 64 + lane;
    const bool valid = p < npairs, spin = g < nspin;
    const int64_t idx = (int64_t)m * npairs + p;
    double x = 0, c2 = 0, p2 = 0, cm = 0, pm = 0;
    int k = 0;
    if (valid) {
        x = pair_z[p];
        c2 = seed2[idx];
        cm = spin ? seedm2[idx] : 0.0;
        k = seedk[idx];
    }
    const int l0 = spin && m < 2 ? 2 : m, lend = spin ? lmax : lmax + EXT_L;
    const double live = spin ? live_spin : live_scalar;
    const Coef64 *cf = coef + alm_base(m, lmax);
    const double *sm = sa + ext_base(m, lmax);
    Ent64 e = {c2, p2, cm, pm};
    int sk = k, sl = l0, res = ENT_SKIP;
    for (int l = l0; l <= lend;) {
        if (wave_any(valid && k == 0 && fmax(fabs(c2), fabs(cm)) >= live)) {
            res = sl;
            break;
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (spin) {
                const Coef64 c = cf[l + t];
                const double u = c.a * x;
                const double n2 = fma(u + c.b, c2, -(c.g * p2));
                const double nm = fma(u - c.b, cm, -(c.g * pm));
                p2 = c2;
                c2 = n2;
                pm = cm;
                cm = nm;
            } else {
                rstep_0(sm[l + t], x, c2, p2);
            }
        }
        l += 2;
        if (k < 0) rescale_slot<FORM_SPIN>(c2, p2, cm, pm, k);
        if (((l - l0) & 7) == 0) {
            e = {c2, p2, cm, pm};
            sk = k;
            sl = l;
        }
    }
    if (valid) {
        ent[idx] = e;
        entk[idx] = sk;
    }
    if (lane == 0) entl[(int64_t)m * ng + g] = res;
}

// ================================================================================================
// prologue / epilogue / weights
// ================================================================================================
// One thread per entry (l, m), l <= lmax + 2, of the scalar form's records: a' and c_l times the stencil's
// coefficients (stencil_in), in FP64.  Bound by HBM: x_E, x_B and the stencil read once (neighbours come
// from the caches), 40 bytes written.  With rsp also the spin form's record.
__global__ __launch_bounds__(256) void k_prologue(const double2 *__restrict__ xE, const double2 *__restrict__ xB,
                                                  const double *__restrict__ kern, const uint32_t *__restrict__ lm,
                                                  const double *__restrict__ sten, const double *__restrict__ sa,
                                                  const double *__restrict__ sc, const Coef64S *__restrict__ cs64,
                                                  int lmax, int64_t nalm, int64_t next, int64_t rec_stride,
                                                  double *__restrict__ rec, SpinRec *__restrict__ rsp)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int rhs = blockIdx.y;
    if (e >= next) return;
    const int l = (int)(lm[e] & 0xffff), m = (int)(lm[e] >> 16);
    const int64_t i = e - (int64_t)EXT_L * m, ns = nalm + ALM_PAD;
    const double2 *pE = xE + rhs * nalm, *pB = xB + rhs * nalm;
    const bool spin = rsp && l <= lmax;
    Coef64S c = {};
    if (spin) c = cs64[i];
    double q[4], K;
    double2 E, B;
    stencil_in(pE, pB, kern, sten, l, m, lmax, nalm, i, q, K, E, B);
    double *r = rec + (rhs * rec_stride + e) * 5;
    // in the signs of the synthesis (see there)
    const int j = (l - m) & 3;
    const double s = (j & 2) ? -sc[e] : sc[e];
    r[0] = (j & 1) ? -sa[e] : sa[e];
#pragma unroll
    for (int t = 0; t < 4; ++t) r[1 + t] = s * q[t];
    if (spin) {
        E = make_double2(K * E.x, m ? K * E.y : 0.0);
        B = make_double2(K * B.x, m ? K * B.y : 0.0);
        SpinRec o;
        o.a = c.a;
        o.b = c.b;
        o.u0 = c.c * (E.x - B.y);
        o.u1 = c.c * (E.y + B.x);
        o.u2 = c.c * (E.x + B.y);
        o.u3 = c.c * (B.x - E.y);
        rsp[rhs * ns + i] = o;
    }
}

// Workgroup sum of 256 threads' values in a fixed order (deterministic); the result in thread 0.
__device__ __forceinline__ double block_sum256(double s, double *sh)
{
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int q = 128; q > 0; q >>= 1) {
        if ((int)threadIdx.x < q) sh[threadIdx.x] += sh[threadIdx.x + q];
        __syncthreads();
    }
    return sh[0];
}

// Sums of the adjoint's ring-block slabs, E/B combination, harmonic diagonal and + lambda x.  The first
// nrbs slabs hold 2h, -2h (spin form): E = -(2h + -2h) / 2, B = (i / 2) (2h - -2h).  The others hold
// the scalar sums T_1, T_2 in units of mu, and with T = c_l times the slab sums
//   E_l = -(w_2 T_1(l+2) + w_0 T_1(l) + w_-2 T_1(l-2) + i (x_1 T_2(l+1) + x_-1 T_2(l-1))),
//   B_l = -(w_2 T_2(l+2) + w_0 T_2(l) + w_-2 T_2(l-2) - i (x_1 T_1(l+1) + x_-1 T_1(l-1))).
// A workgroup walks tiles of 256 entries (l, m) that overlap by two on each side: every thread sums
// the slabs of its entry into LDS and the inner 252 apply the stencil from there, so the slabs, the
// bulk of the traffic, are read once.  Ring blocks that started above l wrote nothing for it.
// With dot_red, also the workgroup partials of the full-m inner product <x, out> (one per workgroup,
// summed in a fixed order by the CG scalar kernel).  blockIdx.y picks one of the right-hand sides of a
// batched group (strides part_stride, v_stride and 2 CG_RED_BLOCKS, lambda la.lam).
constexpr int EPI_TILE = 256 - 2 * EXT_L;
template <typename S>
__global__ __launch_bounds__(256) void k_epilogue(const S *__restrict__ part, const int *__restrict__ wgstart,
                                                  int nrbs, int nrb, int64_t nalm, int64_t next,
                                                  const uint32_t *__restrict__ lm, const double *__restrict__ sten,
                                                  const double *__restrict__ sc, int lmax,
                                                  const double *__restrict__ kern, EpiLam la,
                                                  const double *__restrict__ xE, const double *__restrict__ xB,
                                                  double *__restrict__ outE, double *__restrict__ outB, int proj,
                                                  double *__restrict__ dot_red, int64_t part_stride,
                                                  int64_t v_stride)
{
    __shared__ double sh[256];
    __shared__ double T[4][256];
    const int rhs = blockIdx.y;
    const double lam = la.lam[rhs];
    part += rhs * part_stride;
    outE += rhs * v_stride;
    outB += rhs * v_stride;
    if (xE) {
        xE += rhs * v_stride;
        xB += rhs * v_stride;
    }
    if (dot_red) dot_red += (int64_t)rhs * 2 * CG_RED_BLOCKS;
    const int tid = threadIdx.x;
    const int64_t ns = nalm + ALM_PAD;
    double dot = 0.0;
    for (int64_t e0 = (int64_t)blockIdx.x * EPI_TILE; e0 < next; e0 += (int64_t)gridDim.x * EPI_TILE) {
        const int64_t e = e0 + tid - EXT_L;
        const bool valid = e >= 0 && e < next;
        const uint32_t v = valid ? lm[e] : 0;
        const int l = (int)(v & 0xffff), m = (int)(v >> 16);
        const int64_t i = e - (int64_t)EXT_L * m;
        const int *ws = wgstart + (int64_t)m * nrb;
        const bool inner = valid && tid >= EXT_L && tid < 256 - EXT_L && l <= lmax;
        // everything an entry needs is on its way before the first slab is waited for
        const double s = valid ? sc[e] : 0.0;
        double w[STENCIL] = {}, x[4] = {}, K = 1.0;
        if (inner) {
#pragma unroll
            for (int row = 0; row < STENCIL; ++row) w[row] = sten[row * ns + i];
            if (kern) K = kern[l];
            if (xE) {
                x[0] = xE[2 * i];
                x[1] = xE[2 * i + 1];
                x[2] = xB[2 * i];
                x[3] = xB[2 * i + 1];
            }
        }
        // sum of the slabs [r0, r1) at entry k, two in flight (four: 111 registers against 83 and 4 to 6 % longer where
        // the slabs are many, 16 right-hand sides at Nside 1024 1.34 against 1.28 ms)
        auto slabs = [&](int r0, int r1, int64_t k, double (&t)[4]) {
            for (int rb = r0; rb < r1; rb += 2) {
                bool on[2];
                S q[2][4] = {};
#pragma unroll
                for (int u = 0; u < 2; ++u) on[u] = rb + u < r1 && l >= ws[rb + u];
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (on[u]) {
                        const S *p = part + ((int64_t)(rb + u) * next + k) * 4;
#pragma unroll
                        for (int c = 0; c < 4; ++c) q[u][c] = p[c];
                    }
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int c = 0; c < 4; ++c) t[c] += (double)q[u][c];
            }
        };
        double t[4] = {0, 0, 0, 0}, sp[4] = {0, 0, 0, 0};
        if (valid) slabs(nrbs, nrb, e, t);
        if (inner && l >= 2) slabs(0, nrbs, i, sp);
#pragma unroll
        for (int c = 0; c < 4; ++c) T[c][tid] = s * t[c];
        __syncthreads();
        if (inner) {
            double eR = 0, eI = 0, bR = 0, bI = 0;
            if (l >= 2) {
                auto even = [&](int d, int row) {
                    if (l + d < m) return;
                    eR = fma(-w[row], T[0][tid + d], eR);
                    eI = fma(-w[row], T[1][tid + d], eI);
                    bR = fma(-w[row], T[2][tid + d], bR);
                    bI = fma(-w[row], T[3][tid + d], bI);
                };
                auto odd = [&](int d, int row) {
                    if (l + d < m) return;
                    eR = fma(w[row], T[3][tid + d], eR);
                    eI = fma(-w[row], T[2][tid + d], eI);
                    bR = fma(-w[row], T[1][tid + d], bR);
                    bI = fma(w[row], T[0][tid + d], bI);
                };
                if (nrb > nrbs) {
                    even(-2, ST_WM2);
                    odd(-1, ST_XM1);
                    even(0, ST_W0);
                    odd(1, ST_X1);
                    even(2, ST_W2);
                }
                if (nrbs) {
                    eR -= 0.5 * (sp[0] + sp[2]);
                    eI -= 0.5 * (sp[1] + sp[3]);
                    bR -= 0.5 * (sp[1] - sp[3]);
                    bI += 0.5 * (sp[0] - sp[2]);
                }
            }
            if (m == 0) eI = bI = 0.0;
            eR *= K; eI *= K; bR *= K; bI *= K;
            if (xE) {
                eR += lam * x[0];
                bR += lam * x[2];
                if (m) {
                    eI += lam * x[1];
                    bI += lam * x[3];
                }
            }
            // block systems: the output block of the unknowns held at zero is zero
            if (proj == 1) bR = bI = 0.0;
            if (proj == 2) eR = eI = 0.0;
            outE[2 * i] = eR;
            outE[2 * i + 1] = eI;
            outB[2 * i] = bR;
            outB[2 * i + 1] = bI;
            if (xE) dot += (m ? 2.0 : 1.0) * ((eR * x[0] + eI * x[1]) + (bR * x[2] + bI * x[3]));
        }
        __syncthreads();
    }
    if (dot_red) {
        const double t = block_sum256(dot, sh);
        if (tid == 0) dot_red[blockIdx.x] = t;
    }
}

// W = mask * ninv; block partials of sum(M N^-1), sum(M), #non-finite, #negative, sum over all pixels
__global__ void k_weights(const double *__restrict__ ninv, const uint8_t *__restrict__ mask, double *__restrict__ W,
                          int64_t npix, int ncount, double *__restrict__ red)
{
    // right-hand side rhs takes the N^-1 map rhs mod ncount
    const int rhs = blockIdx.y;
    const int64_t nofs = (int64_t)(rhs % ncount) * npix;
    __shared__ double sh[5][256];
    double a = 0, b = 0, c = 0, d = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < npix; i += (int64_t)gridDim.x * blockDim.x) {
        const double v = ninv[nofs + i];
        const bool obs = mask[i] != 0;
        if (!isfinite(v)) c += 1;
        if (v < 0) d += 1;
        const double w = obs ? v : 0.0;
        W[rhs * npix + i] = w;
        a += w;
        b += obs ? 1.0 : 0.0;
    }
    sh[0][threadIdx.x] = a;
    sh[1][threadIdx.x] = b;
    sh[2][threadIdx.x] = c;
    sh[3][threadIdx.x] = d;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int q = 0; q < 4; ++q) sh[q][threadIdx.x] += sh[q][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 4; ++q) red[((int64_t)rhs * gridDim.x + blockIdx.x) * 4 + q] = sh[q][0];
}

// ================================================================================================
// Ring stage.  One workgroup per ring of N pixels.  Synthesis direction: fold F(m), |m| <= lmax,
// into the N bins (phase e^{i m phi0}), inverse DFT -> gamma at the pixels.  Adjoint direction:
// weight, forward DFT, unfold into every |m| <= lmax (phase e^{-i m phi0}) and multiply by the pixel
// area.  Three kernels cover the rings: a radix-8 FFT of the whole ring in LDS when N is a power of
// two, Bluestein's chirp-z over the whole ring when its convolution (a power-of-two length
// M >= 2N - 1) fits in LDS, else two interleaved sub-transforms of length N / 2, each by Bluestein.
// ================================================================================================
// e^{-i pi n^2 / L}
template <typename T> __device__ __forceinline__ cplx<T> chirp(int n, int L)
{
    return cconj<T>(cis_pi<T>(((int64_t)n * n) % (2 * (int64_t)L), L));
}

// Forward DFT of length L: y_k = sum_n x_n e^{-2 pi i n k / L}; x_n = get(u) for n = tid + NT u,
// y_k delivered as put(u, y) for k = tid + NT u (NT threads, L <= NT NU).
template <typename T, int NT = RT, int NU = RU, class Get, class Put>
__device__ __forceinline__ void dft_forward(cplx<T> *buf, const cplx<T> *bhat, int L, int M, int logM, bool blu,
                                            const cplx<T> *__restrict__ tw, int twn, Get &&get, Put &&put)
{
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int n = tid + NT * u;
        if (n < L) {
            cplx<T> v = get(u);
            if (blu) v = cmul<T>(v, chirp<T>(n, L));
            buf[pd(brev(n, logM))] = v;
        }
    }
    for (int n = L + tid; n < M; n += NT) buf[pd(brev(n, logM))] = mk<T>(0, 0);
    __syncthreads();
    fft_dit<T, NT>(buf, M, tw, twn, -1);
    if (blu) {
        for (int n = tid; n < M; n += NT) buf[pd(n)] = cmul<T>(buf[pd(n)], bhat[n]);
        __syncthreads();
        fft_dif<T, NT>(buf, M, tw, twn, +1);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int kk = tid + NT * u;
            if (kk < L) put(u, cmul<T>(buf[pd(brev(kk, logM))], chirp<T>(kk, L)));
        }
    } else {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int kk = tid + NT * u;
            if (kk < L) put(u, buf[pd(kk)]);
        }
    }
    __syncthreads();
}

// Ring kernels.  MODE 0: F -> maps (o1, o2).  MODE 1: maps (g1, g2) x W -> G.  MODE 2: F -> maps x W -> G
// in place.  MODE 3 (gradient of the solve): F = Y K x as maps px; with o1, o2 holding q = Y K u, per
// pixel  o3 = M (omega q . (g - px) - c),   (o1, o2) = omega W q.
// ================================================================================================
// Ring stage for rings whose length N is a power of two (the equatorial belt when Nside is one):
// the length-N transforms run directly in LDS, one workgroup of RF threads per ring.  F is folded
// and G unfolded in m order, so neighbouring threads read and write neighbouring entries of the
// ring's row; each direction is one FFT of radix-8 passes (floor(log2 N / 3) of them, plus one
// radix-2 or radix-4 step for the remainder), both directions taking natural input to bit-reversed
// output.
// MODE as above.
// ================================================================================================
constexpr int RF = 1024;  // threads per ring workgroup
constexpr int RFU = 8;    // elements per thread: N <= RF * RFU

// Short rings (many orders per bin: 2 lmax + 1 > 8 N): the fold and the unfold run over the orders
// with the whole workgroup instead of one thread per bin.  Thread tau < Q N (Q = floor(RF / N)) takes
// the orders m = tau - lmax + Q N u, which all fall into one bin, sums them in order, and the Q
// partial sums of a bin are added in a fixed tree in LDS.  The unfold gives every order its own
// thread.  Both read and write F / G in m order, neighbouring threads on neighbouring entries.
__device__ __forceinline__ bool short_ring(int N, int lmax) { return 2 * lmax + 1 > 8 * N; }

// X_b = e^{i pi b shift / N} sum_{m = b + N t, |m| <= lmax} (-1)^{t shift} F(m) into buf[pd(b)], b < N;
// buf must hold RF complex entries; ends with a barrier
template <typename T>
__device__ void fold_short(const cplx<T> *__restrict__ F, cplx<T> *buf, int N, int shift, int lmax)
{
    const int tid = threadIdx.x, Q = RF / N, RFp = Q * N;
    if (tid < RFp) {
        const int r = tid - (tid / N) * N;
        const int b = ((r - lmax) % N + N) % N;             // bin of every order of this thread
        int t = (tid - lmax - b) / N;                         // m = b + N t for m = tid - lmax
        const bool flip = shift && (Q & 1);                   // t advances by Q per step
        bool neg = shift && (t & 1);
        T sr = 0, si = 0;
        for (int mm = tid; mm <= 2 * lmax; mm += RFp) {
            const int m = mm - lmax;
            const cplx<T> f = (m >= 0) ? F[2 * m] : F[2 * (-m) + 1];
            sr += neg ? -f.x : f.x;
            si += neg ? -f.y : f.y;
            neg ^= flip;
        }
        buf[tid] = mk<T>(sr, si);
    }
    for (int st = 1; st < Q; st <<= 1) {
        __syncthreads();
        if (tid < RFp) {
            const int q = tid / N;
            if ((q % (2 * st)) == 0 && q + st < Q) buf[tid] = cadd<T>(buf[tid], buf[tid + st * N]);
        }
    }
    __syncthreads();
    cplx<T> x = mk<T>(0, 0);
    int b = 0;
    if (tid < N) {
        b = ((tid - lmax) % N + N) % N;
        x = buf[tid];
        if (shift) x = cmul<T>(x, to_t<T>(cis_pi<double>(b, N)));
    }
    __syncthreads();
    if (tid < N) buf[pd(b)] = x;
    __syncthreads();
}

// G(m) = (-1)^{t shift} e^{-i pi b shift / N} Y_b for every |m| <= lmax, m = b + N t, from Y_b in
// buf[pd(b)] (already scaled); G(0) goes to both components
template <typename T>
__device__ void unfold_short(cplx<T> *__restrict__ G, cplx<T> *buf, int N, int shift, int lmax)
{
    const int tid = threadIdx.x;
    if (shift) {
        for (int b = tid; b < N; b += RF) buf[pd(b)] = cmul<T>(buf[pd(b)], to_t<T>(cis_pi<double>(-b, N)));
        __syncthreads();
    }
    for (int mm = tid; mm <= 2 * lmax; mm += RF) {
        const int m = mm - lmax;
        const int b = ((m % N) + N) % N, t = (m - b) / N;
        cplx<T> g = buf[pd(b)];
        if (shift && (t & 1)) g = mk<T>(-g.x, -g.y);
        if (m > 0) G[2 * m] = g;
        else if (m < 0) G[2 * (-m) + 1] = g;
        else {
            G[0] = g;
            G[1] = g;
        }
    }
}

template <typename T, int MODE>
__device__ __forceinline__ void ring_full_body(cplx<T> *__restrict__ buf, int r, int rhs, cplx<T> *__restrict__ FG,
                                               int64_t fg_stride, const double *__restrict__ g1,
                                               const double *__restrict__ g2, double *__restrict__ o1,
                                               double *__restrict__ o2, int64_t map_stride,
                                               const double *__restrict__ Wt, const RingInfo *__restrict__ rings,
                                               const cplx<T> *__restrict__ tw, int twn, int lmax, double omega,
                                               double *__restrict__ o3, const uint8_t *__restrict__ mask,
                                               const double *__restrict__ cdev)
{
    const RingInfo ri = rings[r];
    const int N = ri.nphi, shift = ri.shift;
    const int logN = 31 - __builtin_clz(N);
    cplx<T> *F = FG + rhs * fg_stride + (int64_t)r * (lmax + 1) * 2;
    const int tid = threadIdx.x;
    const int64_t pofs = rhs * map_stride + ri.ofs;
    const float rN = 1.0f / (float)N;
    cplx<T> v[RFU];

    const bool shortr = short_ring(N, lmax);
    if (MODE != 1) {
        // bin b collects F(m) e^{i m phi0} over m = b + N t, |m| <= lmax (phi0 = pi shift / N)
        if (shortr) {
            fold_short<T>(F, buf, N, shift, lmax);
        } else {
            PhaseSeq ph(tid, RF, N);  // e^{i pi b / N}
#pragma unroll
            for (int u = 0; u < RFU; ++u) {
                const int b = tid + RF * u;
                const double2 e = ph.next();
                if (b < N) buf[pd(b)] = fold_bin_ph<T>(F, b, N, rN, shift, lmax, e);
            }
            __syncthreads();
        }
        fft_dif<T, RF>(buf, N, tw, twn, +1);  // gamma_j = sum_b X_b e^{+2 pi i b j / N}, at brev(j)
#pragma unroll
        for (int u = 0; u < RFU; ++u) {
            const int j = tid + RF * u;
            if (j < N) v[u] = buf[pd(brev(j, logN))];
        }
        __syncthreads();
    }
    if (MODE == 0) {
#pragma unroll
        for (int u = 0; u < RFU; ++u) {
            const int j = tid + RF * u;
            if (j >= N) continue;
            o1[pofs + j] = (double)v[u].x;
            o2[pofs + j] = (double)v[u].y;
        }
        return;
    }
    if (MODE == 3) {
        const double c = *cdev;
#pragma unroll
        for (int u = 0; u < RFU; ++u) {
            const int j = tid + RF * u;
            if (j >= N) continue;
            const int64_t pix = pofs + j;
            const int64_t pm = ri.ofs + j;  // the mask is shared by all right-hand sides
            const double q1 = o1[pix], q2 = o2[pix];
            const double r1 = g1[pix] - (double)v[u].x, r2 = g2[pix] - (double)v[u].y;
            o3[pix] = mask[pm] ? omega * (q1 * r1 + q2 * r2) - c : 0.0;
            const double w = omega * Wt[pix];
            o1[pix] = w * q1;
            o2[pix] = w * q2;
        }
        return;
    }
    // h_j = W_j gamma_j (MODE 2) or W_j (g1 + i g2)_j (MODE 1), in natural order
#pragma unroll
    for (int u = 0; u < RFU; ++u) {
        const int j = tid + RF * u;
        if (j >= N) continue;
        const int64_t pix = pofs + j;
        if (MODE == 1) {
            const T w = Wt ? (T)Wt[pix] : (T)1;
            buf[pd(j)] = mk<T>((T)g1[pix] * w, (T)g2[pix] * w);
        } else {
            buf[pd(j)] = cscale<T>(v[u], (T)Wt[pix]);
        }
    }
    __syncthreads();
    fft_dif<T, RF>(buf, N, tw, twn, -1);  // Y_b = sum_j h_j e^{-2 pi i b j / N}, at brev(b)
    const T om = (T)omega;
    if (shortr) {
        // bins to natural order, scaled (read all, then write: the two orders overlap)
#pragma unroll
        for (int u = 0; u < RFU; ++u) {
            const int b = tid + RF * u;
            if (b < N) v[u] = cscale<T>(buf[pd(brev(b, logN))], om);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < RFU; ++u) {
            const int b = tid + RF * u;
            if (b < N) buf[pd(b)] = v[u];
        }
        __syncthreads();
        unfold_short<T>(F, buf, N, shift, lmax);
        return;
    }
    PhaseSeq ph(tid, RF, N);
#pragma unroll
    for (int u = 0; u < RFU; ++u) {
        const int b = tid + RF * u;
        const double2 e = ph.next();
        if (b < N) unfold_bin_ph<T>(F, b, N, rN, shift, lmax, cscale<T>(buf[pd(brev(b, logN))], om), e);
    }
}

// ================================================================================================
// Ring stage for rings of any length N whose Bluestein convolution (length M >= 2N - 1, a power of
// two) fits in LDS: one DFT of the whole ring per direction by Bluestein's chirp-z, with the chirp
// spectrum of length N from the plan's table; fold and unfold in m order as in ring_full_body.
// MODE as above.
// ================================================================================================
constexpr int RBU = 4;  // elements per thread: N <= RF * RBU

template <typename T, int MODE>
__device__ __forceinline__ void ring_bfull_body(cplx<T> *__restrict__ buf, int r, int rhs, cplx<T> *__restrict__ FG,
                                                int64_t fg_stride, const double *__restrict__ g1,
                                                const double *__restrict__ g2, double *__restrict__ o1,
                                                double *__restrict__ o2, int64_t map_stride,
                                                const double *__restrict__ Wt, const RingInfo *__restrict__ rings,
                                                const cplx<T> *__restrict__ tw, int twn, int lmax, double omega,
                                                double *__restrict__ o3, const uint8_t *__restrict__ mask,
                                                const double *__restrict__ cdev, const cplx<T> *__restrict__ bhat_all)
{
    const RingInfo ri = rings[r];
    const int N = ri.nphi, shift = ri.shift, M = ri.M;
    const int logM = 31 - __builtin_clz(M);
    const cplx<T> *bhat = bhat_all + ri.bofs;
    cplx<T> *F = FG + rhs * fg_stride + (int64_t)r * (lmax + 1) * 2;
    const int tid = threadIdx.x;
    const int64_t pofs = rhs * map_stride + ri.ofs;
    const float rN = 1.0f / (float)N;
    cplx<T> v[RBU];

    const bool shortr = short_ring(N, lmax);
    if (MODE != 1) {
        // gamma_j = sum_b X_b e^{+2 pi i b j / N} = conj(DFT(conj X))_j; get and put run in u order
        if (shortr) {
            fold_short<T>(F, buf, N, shift, lmax);
#pragma unroll
            for (int u = 0; u < RBU; ++u) {
                const int b = tid + RF * u;
                v[u] = b < N ? buf[pd(b)] : mk<T>(0, 0);
            }
            __syncthreads();
            dft_forward<T, RF, RBU>(
                buf, bhat, N, M, logM, true, tw, twn, [&](int u) { return cconj<T>(v[u]); },
                [&](int u, cplx<T> y) { v[u] = cconj<T>(y); });
        } else {
            PhaseSeq ph(tid, RF, N);  // e^{i pi b / N} along b = tid + RF u
            dft_forward<T, RF, RBU>(
                buf, bhat, N, M, logM, true, tw, twn,
                [&](int u) {
                    const double2 e = ph.next();
                    return cconj<T>(fold_bin_ph<T>(F, tid + RF * u, N, rN, shift, lmax, e));
                },
                [&](int u, cplx<T> y) { v[u] = cconj<T>(y); });
        }
    }
    if (MODE == 0) {
#pragma unroll
        for (int u = 0; u < RBU; ++u) {
            const int j = tid + RF * u;
            if (j >= N) continue;
            o1[pofs + j] = (double)v[u].x;
            o2[pofs + j] = (double)v[u].y;
        }
        return;
    }
    if (MODE == 3) {
        const double c = *cdev;
#pragma unroll
        for (int u = 0; u < RBU; ++u) {
            const int j = tid + RF * u;
            if (j >= N) continue;
            const int64_t pix = pofs + j;
            const int64_t pm = ri.ofs + j;  // the mask is shared by all right-hand sides
            const double q1 = o1[pix], q2 = o2[pix];
            const double r1 = g1[pix] - (double)v[u].x, r2 = g2[pix] - (double)v[u].y;
            o3[pix] = mask[pm] ? omega * (q1 * r1 + q2 * r2) - c : 0.0;
            const double w = omega * Wt[pix];
            o1[pix] = w * q1;
            o2[pix] = w * q2;
        }
        return;
    }
#pragma unroll
    for (int u = 0; u < RBU; ++u) {
        const int j = tid + RF * u;
        if (j >= N) continue;
        const int64_t pix = pofs + j;
        if (MODE == 1) {
            const T w = Wt ? (T)Wt[pix] : (T)1;
            v[u] = mk<T>((T)g1[pix] * w, (T)g2[pix] * w);
        } else {
            v[u] = cscale<T>(v[u], (T)Wt[pix]);
        }
    }
    const T om = (T)omega;
    if (shortr) {
        dft_forward<T, RF, RBU>(
            buf, bhat, N, M, logM, true, tw, twn, [&](int u) { return v[u]; },
            [&](int u, cplx<T> y) { v[u] = cscale<T>(y, om); });
#pragma unroll
        for (int u = 0; u < RBU; ++u) {
            const int b = tid + RF * u;
            if (b < N) buf[pd(b)] = v[u];
        }
        __syncthreads();
        unfold_short<T>(F, buf, N, shift, lmax);
        return;
    }
    PhaseSeq ph(tid, RF, N);
    dft_forward<T, RF, RBU>(
        buf, bhat, N, M, logM, true, tw, twn, [&](int u) { return v[u]; },
        [&](int u, cplx<T> y) {
            const double2 e = ph.next();
            unfold_bin_ph<T>(F, tid + RF * u, N, rN, shift, lmax, cscale<T>(y, om), e);
        });
}

// The whole-ring LDS kernels in one launch: the first nbf workgroups of the grid take a Bluestein ring each
// (the longer ones), the others a power-of-two ring.
template <typename T, int MODE>
__global__ __launch_bounds__(RF) void k_ring_lds(cplx<T> *__restrict__ FG, int64_t fg_stride, RingArgs a,
                                                 int64_t map_stride, const RingInfo *__restrict__ rings,
                                                 const int *__restrict__ order_bf, int nbf,
                                                 const int *__restrict__ order_p2, const cplx<T> *__restrict__ tw,
                                                 int twn, int lmax, double omega, const cplx<T> *__restrict__ bhat_all)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cplx<T> *buf = reinterpret_cast<cplx<T> *>(smem_raw);
    const int b = blockIdx.x;
    if (b < nbf)
        ring_bfull_body<T, MODE>(buf, order_bf[b], blockIdx.y, FG, fg_stride, a.g1, a.g2, a.o1, a.o2, map_stride, a.W,
                                 rings, tw, twn, lmax, omega, a.o3, a.mask, a.cdev, bhat_all);
    else
        ring_full_body<T, MODE>(buf, order_p2[b - nbf], blockIdx.y, FG, fg_stride, a.g1, a.g2, a.o1, a.o2, map_stride,
                                a.W, rings, tw, twn, lmax, omega, a.o3, a.mask, a.cdev);
}

// ================================================================================================
// Ring stage for the remaining rings (whole-ring convolution too long for LDS): the length-N DFT
// (N even) splits into two interleaved sub-DFTs of length L = N / 2 over the even and odd bins, each
// by Bluestein with the chirp spectrum of length L; the radix-2 step in registers combines them:
//   synthesis  gamma[j1] = Y0[j1] + w^j1 Y1[j1],  gamma[j1 + L] = Y0[j1] - w^j1 Y1[j1],  w = e^{2 pi i/N}
//   adjoint    u_q[j1] = w^{-q j1} (h[j1] + (-1)^q h[j1 + L]),  bins 2 k + q = DFT_L(u_q)[k].
// MODE as above.
// ================================================================================================
template <typename T, int MODE>
__global__ __launch_bounds__(RF) void k_ring_b2(cplx<T> *__restrict__ FG, int64_t fg_stride,
                                                const double *__restrict__ g1, const double *__restrict__ g2,
                                                double *__restrict__ o1, double *__restrict__ o2, int64_t map_stride,
                                                const double *__restrict__ Wt, const RingInfo *__restrict__ rings,
                                                const int *__restrict__ order, const cplx<T> *__restrict__ tw,
                                                int twn, int lmax, double omega, double *__restrict__ o3,
                                                const uint8_t *__restrict__ mask, const double *__restrict__ cdev,
                                                const cplx<T> *__restrict__ bhat_all)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cplx<T> *buf = reinterpret_cast<cplx<T> *>(smem_raw);
    const int r = order[blockIdx.x];
    const int rhs = blockIdx.y;
    const RingInfo ri = rings[r];
    const int N = ri.nphi, L = N / 2, shift = ri.shift, M = ri.M;
    const int logM = 31 - __builtin_clz(M);
    const cplx<T> *bhat = bhat_all + ri.bofs;
    cplx<T> *F = FG + rhs * fg_stride + (int64_t)r * (lmax + 1) * 2;
    const int tid = threadIdx.x;
    const int64_t pofs = rhs * map_stride + ri.ofs;
    const float rN = 1.0f / (float)N;
    cplx<T> v[RBU][2];

    if (MODE != 1) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            // Y_q = inverse DFT_L of the bins 2 k + q; get and put run in u order
            PhaseSeq ph(2 * tid + q, 2 * RF, N);  // e^{i pi b / N} along b = 2 (tid + RF u) + q
            dft_forward<T, RF, RBU>(
                buf, bhat, L, M, logM, true, tw, twn,
                [&](int u) {
                    const double2 e = ph.next();
                    return cconj<T>(fold_bin_ph<T>(F, 2 * (tid + RF * u) + q, N, rN, shift, lmax, e));
                },
                [&](int u, cplx<T> y) { v[u][q] = cconj<T>(y); });
        }
        PhaseSeq pw(2 * tid, 2 * RF, N);  // e^{2 pi i j1 / N}
#pragma unroll
        for (int u = 0; u < RBU; ++u) {
            const int j1 = tid + RF * u;
            const double2 w = pw.next();
            if (j1 >= L) continue;
            const cplx<T> t = cmul<T>(to_t<T>(w), v[u][1]), a = v[u][0];
            v[u][0] = cadd<T>(a, t);
            v[u][1] = csub<T>(a, t);
        }
    }
    if (MODE == 0) {
#pragma unroll
        for (int u = 0; u < RBU; ++u) {
            const int j1 = tid + RF * u;
            if (j1 >= L) continue;
#pragma unroll
            for (int j2 = 0; j2 < 2; ++j2) {
                o1[pofs + j1 + L * j2] = (double)v[u][j2].x;
                o2[pofs + j1 + L * j2] = (double)v[u][j2].y;
            }
        }
        return;
    }
    if (MODE == 3) {
        const double c = *cdev;
#pragma unroll
        for (int u = 0; u < RBU; ++u) {
            const int j1 = tid + RF * u;
            if (j1 >= L) continue;
#pragma unroll
            for (int j2 = 0; j2 < 2; ++j2) {
                const int64_t pix = pofs + j1 + L * j2;
                const int64_t pm = ri.ofs + j1 + L * j2;  // the mask is shared by all right-hand sides
                const double q1 = o1[pix], q2 = o2[pix];
                const double r1 = g1[pix] - (double)v[u][j2].x, r2 = g2[pix] - (double)v[u][j2].y;
                o3[pix] = mask[pm] ? omega * (q1 * r1 + q2 * r2) - c : 0.0;
                const double w = omega * Wt[pix];
                o1[pix] = w * q1;
                o2[pix] = w * q2;
            }
        }
        return;
    }
    PhaseSeq pw(2 * tid, 2 * RF, N);
#pragma unroll
    for (int u = 0; u < RBU; ++u) {
        const int j1 = tid + RF * u;
        const double2 w = pw.next();
        if (j1 >= L) continue;
#pragma unroll
        for (int j2 = 0; j2 < 2; ++j2) {
            const int64_t pix = pofs + j1 + L * j2;
            if (MODE == 1) {
                const T wt = Wt ? (T)Wt[pix] : (T)1;
                v[u][j2] = mk<T>((T)g1[pix] * wt, (T)g2[pix] * wt);
            } else {
                v[u][j2] = cscale<T>(v[u][j2], (T)Wt[pix]);
            }
        }
        const cplx<T> h0 = v[u][0], h1 = v[u][1];
        v[u][0] = cadd<T>(h0, h1);
        v[u][1] = cmul<T>(cconj<T>(to_t<T>(w)), csub<T>(h0, h1));
    }
    const T om = (T)omega;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        PhaseSeq pf(2 * tid + q, 2 * RF, N);  // put runs in u order
        dft_forward<T, RF, RBU>(
            buf, bhat, L, M, logM, true, tw, twn, [&](int u) { return v[u][q]; },
            [&](int u, cplx<T> y) {
                const double2 e = pf.next();
                unfold_bin_ph<T>(F, 2 * (tid + RF * u) + q, N, rN, shift, lmax, cscale<T>(y, om), e);
            });
    }
}

// ================================================================================================
// vector kernels (FP64): full-m inner product and the CG updates
// ================================================================================================
constexpr int RED_BLOCKS = 512;

__global__ void k_dot_part(const double *__restrict__ a, const double *__restrict__ b, int64_t n, int64_t nalm, int lmax,
                           double *__restrict__ red)
{
    __shared__ double sh[256];
    double s = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double w = ((i % nalm) <= lmax) ? 1.0 : 2.0;
        s += w * (a[2 * i] * b[2 * i] + a[2 * i + 1] * b[2 * i + 1]);
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int q = 128; q > 0; q >>= 1) {
        if ((int)threadIdx.x < q) sh[threadIdx.x] += sh[threadIdx.x + q];
        __syncthreads();
    }
    if (threadIdx.x == 0) red[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(256) void k_sum_part(const double *__restrict__ red, int n, int stride, int ncomp,
                                                  double *__restrict__ out)
{
    // deterministic: per component, thread t sums the block partials t, t + 256, ... in order, then
    // a fixed tree over the threads
    __shared__ double sh[256];
    for (int c = 0; c < ncomp; ++c) {
        double s = 0;
        for (int i = threadIdx.x; i < n; i += 256) s += red[(int64_t)i * stride + c];
        const double t = block_sum256(s, sh);
        if (threadIdx.x == 0) out[c] = t;
        __syncthreads();
    }
}

// Fixed-order sum of n workgroup partials by one workgroup of 256 threads (thread t sums partials
// t, t + 256, ... in order, then a tree), the total in thread 0
__device__ __forceinline__ double sum_partials256(const double *__restrict__ red, int n, double *sh)
{
    double s = 0.0;
    for (int j = threadIdx.x; j < n; j += 256) s += red[j];
    return block_sum256(s, sh);
}

// The vector half of a PCG iteration, one right-hand side of the list per blockIdx.y: x += alpha p,
// r -= alpha w and the partials of <r, r>.  Every workgroup sums the <p, w> partials in the same fixed
// order and forms alpha itself (0 on breakdown, which raises the flag); the first one leaves the
// scalars.  Bound by HBM, 96 bytes per coefficient; at small sizes by the launch, which the right-hand
// sides of a batch share.
__global__ __launch_bounds__(256) void k_cg_xr_alpha(double2 *__restrict__ x, double2 *__restrict__ r,
                                                     const double2 *__restrict__ p, const double2 *__restrict__ w,
                                                     double *__restrict__ red, int n_red, double *__restrict__ scal,
                                                     int *__restrict__ flag, int64_t nc, int64_t nalm, int lmax,
                                                     CgList L)
{
    __shared__ double sh[256];
    const int q = L.rhs[blockIdx.y];
    x += q * nc;
    r += q * nc;
    p += q * nc;
    w += q * nc;
    red += (int64_t)q * 2 * CG_RED_BLOCKS;
    scal += 8 * q;
    flag += q;
    const double pw = sum_partials256(red, n_red, sh);
    __syncthreads();
    const double rz = scal[0];
    const bool bad = flag[0] != 0 || !(pw > 0.0) || !isfinite(pw);
    const double a = bad ? 0.0 : rz / pw;
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += (int64_t)gridDim.x * blockDim.x) {
        const double2 pi = p[i], wi = w[i];
        double2 xi = x[i], ri = r[i];
        xi.x = fma(a, pi.x, xi.x);
        xi.y = fma(a, pi.y, xi.y);
        ri.x = fma(-a, wi.x, ri.x);
        ri.y = fma(-a, wi.y, ri.y);
        x[i] = xi;
        r[i] = ri;
        const double wgt = (i < nalm ? i : i - nalm) <= lmax ? 1.0 : 2.0;  // nc = 2 nalm
        s += wgt * (ri.x * ri.x + ri.y * ri.y);
    }
    const double t = block_sum256(s, sh);
    if (threadIdx.x == 0) {
        red[CG_RED_BLOCKS + blockIdx.x] = t;
        if (blockIdx.x == 0) {
            scal[1] = pw;
            scal[2] = a;
            scal[7] = rz;
            if (bad) flag[0] = 1;
        }
    }
}

// p = P r + beta p with beta = P <r, r> / rz formed the same way from the partials of <r, r>.  What the host
// decides on, <r, r> and the flag, goes to its pinned memory from here (two copies after every iteration
// before: 400 iterations at Nside 32 29.0 -> 26.8 ms)
__global__ __launch_bounds__(256) void k_cg_p_beta(double2 *__restrict__ p, const double2 *__restrict__ r,
                                                   const double *__restrict__ red, int n_red,
                                                   double *__restrict__ scal, int64_t nc, CgList L,
                                                   const int *__restrict__ flag, double *__restrict__ host)
{
    __shared__ double sh[256];
    const int q = L.rhs[blockIdx.y];
    const double pc = L.pc[blockIdx.y];
    p += q * nc;
    r += q * nc;
    scal += 8 * q;
    const double rr = sum_partials256(red + (int64_t)q * 2 * CG_RED_BLOCKS + CG_RED_BLOCKS, n_red, sh);
    const double rz_old = scal[7];
    const double rz = pc * rr;
    const double bt = (rz_old > 0.0) ? rz / rz_old : 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += (int64_t)gridDim.x * blockDim.x) {
        const double2 ri = r[i];
        double2 pi = p[i];
        pi.x = fma(bt, pi.x, pc * ri.x);
        pi.y = fma(bt, pi.y, pc * ri.y);
        p[i] = pi;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        scal[3] = rr;
        scal[4] = bt;
        scal[0] = rz;
        host[2 * q] = rr;
        host[2 * q + 1] = (double)flag[q];
        __threadfence_system();
    }
}

__global__ void k_cg_p(double *__restrict__ p, const double *__restrict__ r, const double *__restrict__ beta,
                       double precond, int64_t n2)
{
    const double bt = *beta;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = fma(bt, p[i], precond * r[i]);
}

__global__ void k_axpby(double *__restrict__ y, double a, const double *__restrict__ x, double b, int64_t n2)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n2; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = a * x[i] + b * y[i];
}

// ================================================================================================
// launchers
// ================================================================================================
bool pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }

void launch_prologue(Plan &P, const double *xE, const double *xB, const double *kern, int nrhs, bool spin)
{
    dim3 g((unsigned)cdiv(P.next, 256), nrhs);
    k_prologue<<<g, 256, 0, P.stream>>>((const double2 *)xE, (const double2 *)xB, kern, P.d_lm, P.d_sten, P.d_sa,
                                        P.d_sc, P.d_coef64s, P.lmax, P.nalm, P.next, P.rec_stride, P.d_rec,
                                        spin ? (SpinRec *)P.d_rec_spin : nullptr);
}

void launch_epilogue_batched(Plan &P, int q, const double *kern, const double *lam, const double *xE,
                             const double *xB, double *outE, double *outB, int64_t v_stride, double *dot_red)
{
    const int n = std::min(NBR, P.nrhs - NBR * q);
    EpiLam la = {};
    for (int r = 0; r < n; ++r) la.lam[r] = lam[r];
    const dim3 g(dot_red ? (unsigned)cg_red_blocks(P) : (unsigned)cdiv(P.next, EPI_TILE), n);
    k_epilogue<float><<<g, 256, 0, P.stream>>>((const float *)P.d_part, P.d_wgstart_b, P.nrbs_b_cur, P.nrb_b_cur,
                                              P.nalm, P.next, P.d_lm, P.d_sten, P.d_sc, P.lmax, kern, la, xE, xB,
                                              outE, outB, P.proj, dot_red, (int64_t)P.nrb_b_cur * P.next * 4,
                                              v_stride);
}

void launch_entry(Plan &P)
{
    const int gpb = (int)cdiv(P.ng64, 4);
    const bool f32 = P.prec == AKRA_FP32;
    k_entry<<<(unsigned)((int64_t)gpb * (P.lmax + 1)), 256, 0, P.stream>>>(
        P.d_seed2, P.d_seedm2, P.d_seedk, P.d_pair_z, P.d_coef64, P.d_sa, P.d_ent, P.d_entk, P.d_entl, P.lmax,
        P.npairs, P.ng64, gpb, P.spin_groups, f32 ? 0x1p-44 : 0x1p-100, f32 ? 0x1p-49 : 0x1p-105);
}

// Legendre synthesis of the prologue's records: every 64-pair group (live false), or the groups of
// the current weights by class (live true)
void launch_leg_synth(Plan &P, bool fp32, int nrhs, bool live)
{
    const GroupSet &G = live && P.skip_rings ? P.gs_live : P.gs_all;
    auto n = [&](int c) { return G.npol[c] + G.nmain[c]; };
    auto two = [&]() {
        if (n(GCLS_BOTH)) leg_synth_cls<GCLS_BOTH>(P, fp32, nrhs, G.list[GCLS_BOTH], G.npol[GCLS_BOTH], G.nmain[GCLS_BOTH]);
    };
    auto one = [&]() {
        if (n(GCLS_NORTH))
            leg_synth_cls<GCLS_NORTH>(P, fp32, nrhs, G.list[GCLS_NORTH], G.npol[GCLS_NORTH], G.nmain[GCLS_NORTH]);
        if (n(GCLS_SOUTH))
            leg_synth_cls<GCLS_SOUTH>(P, fp32, nrhs, G.list[GCLS_SOUTH], G.npol[GCLS_SOUTH], G.nmain[GCLS_SOUTH]);
    };
    // the classes write F of disjoint rings: the two-sided groups on the side stream
    if (P.fork_classes && n(GCLS_BOTH) && n(GCLS_NORTH) + n(GCLS_SOUTH)) fork_join(P, two, one);
    else {
        two();
        one();
    }
}

bool adj_shape_supported(int r, int w, int l)
{
#define AKRA_ADJ_SUP(a, b, c) \
    if (r == a && w == b && l == c) return true;
    AKRA_ADJ_SHAPES(AKRA_ADJ_SUP)
#undef AKRA_ADJ_SUP
    return false;
}

int adj_blocks_spin_total(const Plan &P, bool live)
{
    const GroupSet &G = live && P.skip_rings ? P.gs_live : P.gs_all;
    int n = 0;
    for (int c = 0; c < GCLS_N; ++c) n += adj_blocks_spin(P, c, G.npol[c]);
    return n;
}

int adj_blocks_total(const Plan &P, bool live)
{
    const GroupSet &G = live && P.skip_rings ? P.gs_live : P.gs_all;
    int n = adj_blocks_spin_total(P, live);
    for (int c = 0; c < GCLS_N; ++c) n += adj_blocks_main(P, c, G.nmain[c]);
    return n;
}

// ring blocks of a class: the spin blocks of every class first (two-sided, north, south), then the
// scalar ones in the same order (the slabs are disjoint)
static void adj_first(const Plan &P, const GroupSet &G, int nspin, int cls, int &rbs, int &rbm)
{
    rbs = 0;
    rbm = nspin;
    for (int c = 0; c < cls; ++c) {
        rbs += adj_blocks_spin(P, c, G.npol[c]);
        rbm += adj_blocks_main(P, c, G.nmain[c]);
    }
}

template <int CLS>
static void adj_cls(Plan &P, bool fp32, int rhs, const GroupSet &G, const uint8_t *lv, int nspin, int nrb)
{
    if (G.npol[CLS] + G.nmain[CLS] <= 0) return;
    int rbs, rbm;
    adj_first(P, G, nspin, CLS, rbs, rbm);
    leg_adj_cls<CLS>(P, fp32, rhs, G.list[CLS], G.npol[CLS], G.nmain[CLS], lv, rbs, rbm, nrb);
}

// Legendre adjoint of d_FG (right-hand side rhs) into the partial sums, over every 64-pair group
// (live false) or the groups of the current weights by class, reading only rings that carry weight
// (live true).  The epilogue sums the nrb_cur blocks written, the first nrbs_cur of them in the spin form.
void launch_leg_adj(Plan &P, bool fp32, int rhs, bool live)
{
    live = live && P.skip_rings;
    const GroupSet &G = live ? P.gs_live : P.gs_all;
    const uint8_t *lv = live ? P.d_ring_live : nullptr;
    const int nspin = adj_blocks_spin_total(P, live), nrb = adj_blocks_total(P, live);
    auto n = [&](int c) { return G.npol[c] + G.nmain[c]; };
    auto two = [&]() { adj_cls<GCLS_BOTH>(P, fp32, rhs, G, lv, nspin, nrb); };
    auto one = [&]() {
        adj_cls<GCLS_NORTH>(P, fp32, rhs, G, lv, nspin, nrb);
        adj_cls<GCLS_SOUTH>(P, fp32, rhs, G, lv, nspin, nrb);
    };
    if (P.fork_classes && n(GCLS_BOTH) && n(GCLS_NORTH) + n(GCLS_SOUTH)) fork_join(P, two, one);
    else {
        two();
        one();
    }
    P.nrb_cur = nrb;
    P.nrbs_cur = nspin;
}

int cg_red_blocks(const Plan &P) { return (int)std::min<int64_t>(CG_RED_BLOCKS, cdiv(P.nalm, 256)); }

void launch_epilogue(Plan &P, bool fp32, const double *kern, double lam, const double *xE, const double *xB,
                     double *outE, double *outB, double *dot_red)
{
    const dim3 g(dot_red ? (unsigned)cg_red_blocks(P) : (unsigned)cdiv(P.next, EPI_TILE));
    EpiLam la = {};
    la.lam[0] = lam;
    if (fp32)
        k_epilogue<float><<<g, 256, 0, P.stream>>>((const float *)P.d_part, P.d_wgstart, P.nrbs_cur, P.nrb_cur, P.nalm,
                                                   P.next, P.d_lm, P.d_sten, P.d_sc, P.lmax, kern, la, xE, xB, outE,
                                                   outB, P.proj, dot_red, 0, 0);
    else
        k_epilogue<double><<<g, 256, 0, P.stream>>>((const double *)P.d_part, P.d_wgstart, P.nrbs_cur, P.nrb_cur,
                                                    P.nalm, P.next, P.d_lm, P.d_sten, P.d_sc, P.lmax, kern, la, xE,
                                                    xB, outE, outB, P.proj, dot_red, 0, 0);
}

void launch_cg_xr_alpha(Plan &P, double *x, double *r, const double *p, const double *w, double *scal, int *flag,
                        int64_t n_complex, const CgList &L)
{
    const int nb = cg_red_blocks(P);
    k_cg_xr_alpha<<<dim3(nb, L.n), 256, 0, P.stream>>>((double2 *)x, (double2 *)r, (const double2 *)p,
                                                       (const double2 *)w, P.d_red_cg, nb, scal, flag, n_complex,
                                                       P.nalm, P.lmax, L);
}

void launch_cg_p_beta(Plan &P, double *p, const double *r, double *scal, int64_t n_complex, const CgList &L)
{
    const int nb = cg_red_blocks(P);
    k_cg_p_beta<<<dim3(nb, L.n), 256, 0, P.stream>>>((double2 *)p, (const double2 *)r, P.d_red_cg, nb, scal, n_complex,
                                                     L, P.d_flag, P.h_cg);
}

// The ring kinds of a RingSet: RK_P2 whole power-of-two rings (LDS FFT), RK_BF whole-ring Bluestein,
// RK_BL rings split into two half-length Bluestein transforms, RK_REG + q the register engine's
// lists (see akra_internal.h)
template <typename T, int MODE>
static void ring_launch_t(Plan &P, const RingSet &RS, const double *g1, const double *g2, double *o1, double *o2,
                          const double *W, double *o3, const uint8_t *mask, const double *cdev, int nrhs,
                          bool split = true)
{
    const int64_t fg_stride = (int64_t)P.nrings * (P.lmax + 1) * 2;
    const void *tw = std::is_same<T, double>::value ? P.d_tw64 : P.d_tw32;
    const cplx<T> *bh = (const cplx<T> *)(std::is_same<T, double>::value ? P.d_bhat64 : P.d_bhat32);
    // (a plan without the lists for fewer rings keeps the others in every launch)
    const bool few = RS.n[RK_FEW_P2] + RS.n[RK_FEW_BF] > 0 && (int64_t)P.nrings * nrhs < RING_ENGINE_MIN;
    const int kp = few ? RK_FEW_P2 : RK_P2, kb = few ? RK_FEW_BF : RK_BF;
    if (RS.n[kp] + RS.n[kb]) {
        // power-of-two rings: N = 4 sub <= 4 nside <= 8192 = RF RFU (nside <= 2048 is enforced at plan creation)
        size_t nmax = RF;  // the short-ring fold
        if (RS.n[kp]) nmax = std::max(nmax, 4 * (size_t)P.maxM_p2);
        if (RS.n[kb]) nmax = std::max(nmax, (size_t)P.maxM_bf);
        const size_t sm = sizeof(cplx<T>) * (nmax + nmax / 32);
        k_ring_lds<T, MODE><<<dim3(RS.n[kb] + RS.n[kp], nrhs), RF, sm, P.stream>>>(
            (cplx<T> *)P.d_FG, fg_stride, RingArgs{g1, g2, o1, o2, W, o3, mask, cdev}, P.npix, P.d_rings,
            RS.order[kb], RS.n[kb], RS.order[kp], (const cplx<T> *)tw, P.twn, P.lmax, P.omega, bh);
    }
    if (RS.n[RK_BL]) {
        size_t sm = sizeof(cplx<T>) * (size_t)(P.maxM_bl + P.maxM_bl / 32);
        k_ring_b2<T, MODE><<<dim3(RS.n[RK_BL], nrhs), RF, sm, P.stream>>>(
            (cplx<T> *)P.d_FG, fg_stride, g1, g2, o1, o2, P.npix, W, P.d_rings, RS.order[RK_BL], (const cplx<T> *)tw,
            P.twn, P.lmax, P.omega, o3, mask, cdev, bh);
    }
    if (few) return;  // every whole ring is done; longer transforms than 2048 points have no such plan
    ring16_launch<T, MODE>(P, RS, RingArgs{g1, g2, o1, o2, W, o3, mask, cdev}, nrhs, split);
}

// Spectra of the Bluestein chirps, one per distinct sub-transform length L (plan creation):
//   bhat = FFT_M(b) / M,  b_n = e^{+i pi n^2 / L} for n in (-L, L) (wrapped mod M), in FP64 and, with b32, FP32.
__global__ __launch_bounds__(RT) void k_bhat(const int *__restrict__ Ls, const int *__restrict__ Ms,
                                             const int64_t *__restrict__ ofs, const double2 *__restrict__ tw,
                                             int twn, double2 *__restrict__ b64, float2 *__restrict__ b32)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double2 *buf = reinterpret_cast<double2 *>(smem_raw);
    const int L = Ls[blockIdx.x], M = Ms[blockIdx.x];
    const int64_t o = ofs[blockIdx.x];
    const int logM = 31 - __builtin_clz(M);
    for (int n = threadIdx.x; n < M; n += RT) {
        double2 v = make_double2(0.0, 0.0);
        if (n < L) v = cconj<double>(chirp<double>(n, L));
        else if (n > M - L) v = cconj<double>(chirp<double>(M - n, L));
        buf[pd(brev(n, logM))] = v;
    }
    __syncthreads();
    fft_dit<double>(buf, M, tw, twn, -1);
    const double inv = 1.0 / (double)M;
    for (int n = threadIdx.x; n < M; n += RT) {
        const double2 v = cscale<double>(buf[pd(n)], inv);
        b64[o + n] = v;
        if (b32) b32[o + n] = make_float2((float)v.x, (float)v.y);
    }
}

void launch_bhat_reorder(Plan &P, int logm, const int64_t *src_ofs, const int64_t *dst_ofs, int n)
{
    launch_bhat_reorder_f64(P, logm, src_ofs, dst_ofs, n);
    if (P.prec == AKRA_FP32) launch_bhat_reorder_f32(P, logm, src_ofs, dst_ofs, n);
}

void launch_bhat(Plan &P, const int *Ls, const int *Ms, const int64_t *ofs, int n, int maxM)
{
    k_bhat<<<n, RT, sizeof(double2) * (size_t)(maxM + maxM / 32), P.stream>>>(Ls, Ms, ofs, (const double2 *)P.d_tw64,
                                                                              P.twn, (double2 *)P.d_bhat64,
                                                                              (float2 *)P.d_bhat32);
}

// every ring (live false), or the rings that carry weight in the current weights (live true)
void launch_ring(Plan &P, bool fp32, int mode, const double *g1, const double *g2, double *o1, double *o2,
                 const double *W, int nrhs, bool live)
{
    const RingSet &RS = live && P.skip_rings ? P.rs_live : P.rs_all;
    if (fp32) {
        if (mode == 0) ring_launch_t<float, 0>(P, RS, g1, g2, o1, o2, W, nullptr, nullptr, nullptr, nrhs);
        else if (mode == 1) ring_launch_t<float, 1>(P, RS, g1, g2, o1, o2, W, nullptr, nullptr, nullptr, nrhs);
        else ring_launch_t<float, 2>(P, RS, g1, g2, o1, o2, W, nullptr, nullptr, nullptr, nrhs);
    } else {
        if (mode == 0) ring_launch_t<double, 0>(P, RS, g1, g2, o1, o2, W, nullptr, nullptr, nullptr, nrhs);
        else if (mode == 1) ring_launch_t<double, 1>(P, RS, g1, g2, o1, o2, W, nullptr, nullptr, nullptr, nrhs);
        else ring_launch_t<double, 2>(P, RS, g1, g2, o1, o2, W, nullptr, nullptr, nullptr, nrhs);
    }
}

// Two chains, one per class of ring groups, each running synthesis, ring stage and adjoint of its
// class: the groups weighted on both sides on the side stream, those weighted on one side on the
// plan stream.  A chain's rings are those of its groups, so the chains write F and G of disjoint
// rings and partial sums of disjoint ring blocks; a chain's ring stage needs only its own
// synthesis, and its adjoint only its own rings, so no stage waits for the other class.
void launch_weighted_chains(Plan &P, bool fp32, const double *W)
{
    const GroupSet &G = P.gs_live;
    const uint8_t *lv = P.d_ring_live;
    const int nspin = adj_blocks_spin_total(P, true), nrb = adj_blocks_total(P, true);
    auto n = [&](int c) { return G.npol[c] + G.nmain[c]; };
    auto ring = [&](const RingSet &RS) {
        if (fp32) ring_launch_t<float, 2>(P, RS, nullptr, nullptr, nullptr, nullptr, W, nullptr, nullptr, nullptr, 1, false);
        else ring_launch_t<double, 2>(P, RS, nullptr, nullptr, nullptr, nullptr, W, nullptr, nullptr, nullptr, 1, false);
    };
    auto two = [&]() {
        leg_synth_cls<GCLS_BOTH>(P, fp32, 1, G.list[GCLS_BOTH], G.npol[GCLS_BOTH], G.nmain[GCLS_BOTH]);
        ring(P.rs_cls[0]);
        adj_cls<GCLS_BOTH>(P, fp32, 0, G, lv, nspin, nrb);
    };
    auto one = [&]() {
        if (n(GCLS_NORTH))
            leg_synth_cls<GCLS_NORTH>(P, fp32, 1, G.list[GCLS_NORTH], G.npol[GCLS_NORTH], G.nmain[GCLS_NORTH]);
        if (n(GCLS_SOUTH))
            leg_synth_cls<GCLS_SOUTH>(P, fp32, 1, G.list[GCLS_SOUTH], G.npol[GCLS_SOUTH], G.nmain[GCLS_SOUTH]);
        ring(P.rs_cls[1]);
        adj_cls<GCLS_NORTH>(P, fp32, 0, G, lv, nspin, nrb);
        adj_cls<GCLS_SOUTH>(P, fp32, 0, G, lv, nspin, nrb);
    };
    fork_join(P, two, one);
    P.nrb_cur = nrb;
    P.nrbs_cur = nspin;
}

void launch_ring_grad(Plan &P, const double *g1, const double *g2, double *q1, double *q2, const double *W,
                      double *dninv, const uint8_t *mask, const double *cdev)
{
    ring_launch_t<double, 3>(P, P.rs_all, g1, g2, q1, q2, W, dninv, mask, cdev, 1);
}

// right-hand side of the backward solve: the upstream gradient on the stored (Re, Im) of the alm,
// divided by the full-m weight (1 for m = 0, 2 for m > 0), Im(a_l0) dropped
__global__ void k_vjp_rhs(const double *__restrict__ vE, const double *__restrict__ vB, double *__restrict__ bE,
                          double *__restrict__ bB, int64_t nalm, int lmax)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nalm) return;
    const bool m0 = i <= lmax;
    const double s = m0 ? 1.0 : 0.5;
    bE[2 * i] = s * vE[2 * i];
    bE[2 * i + 1] = m0 ? 0.0 : s * vE[2 * i + 1];
    bB[2 * i] = s * vB[2 * i];
    bB[2 * i + 1] = m0 ? 0.0 : s * vB[2 * i + 1];
}

void launch_vjp_rhs(Plan &P, const double *vE, const double *vB, double *bE, double *bB)
{
    k_vjp_rhs<<<(unsigned)cdiv(P.nalm, 256), 256, 0, P.stream>>>(vE, vB, bE, bB, P.nalm, P.lmax);
}

__global__ void k_scale_scalar(double *out, const double *in, double f) { *out = f * *in; }

void launch_scale_scalar(Plan &P, double *out, const double *in, double f)
{
    k_scale_scalar<<<1, 1, 0, P.stream>>>(out, in, f);
}

// one workgroup per ring: 1 when any of the nrhs weight maps has a nonzero weight on the ring
__global__ __launch_bounds__(256) void k_ring_live(const double *__restrict__ W, const RingInfo *__restrict__ rings,
                                                   int64_t npix, int nrhs, uint8_t *__restrict__ live)
{
    const RingInfo ri = rings[blockIdx.x];
    int any = 0;
    for (int r = 0; r < nrhs; ++r)
        for (int j = threadIdx.x; j < ri.nphi; j += blockDim.x) any |= W[r * npix + ri.ofs + j] != 0.0;
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) live[blockIdx.x] = any ? 1 : 0;
}

void launch_ring_live(Plan &P, int nrhs)
{
    k_ring_live<<<P.nrings, 256, 0, P.stream>>>(P.d_W, P.d_rings, P.npix, nrhs, P.d_ring_live);
}

void launch_weights(Plan &P, const double *ninv, const uint8_t *mask, int nrhs, int ncount)
{
    k_weights<<<dim3(RED_BLOCKS, nrhs), 256, 0, P.stream>>>(ninv, mask, P.d_W, P.npix, ncount, P.d_red);
    for (int r = 0; r < nrhs; ++r)
        k_sum_part<<<1, 256, 0, P.stream>>>(P.d_red + (int64_t)r * RED_BLOCKS * 4, RED_BLOCKS, 4, 4, P.d_scal + 8 + 4 * r);
}

void launch_dot(Plan &P, const double *a, const double *b, double *out_dev, int64_t n_complex)
{
    k_dot_part<<<RED_BLOCKS, 256, 0, P.stream>>>(a, b, n_complex, P.nalm, P.lmax, P.d_red);
    k_sum_part<<<1, 256, 0, P.stream>>>(P.d_red, RED_BLOCKS, 1, 1, out_dev);
}

void launch_cg_p(Plan &P, double *p, const double *r, const double *beta_dev, double precond, int64_t n_complex)
{
    k_cg_p<<<1024, 256, 0, P.stream>>>(p, r, beta_dev, precond, 2 * n_complex);
}

void launch_axpby(Plan &P, double *y, double a, const double *x, double b, int64_t n_complex)
{
    k_axpby<<<1024, 256, 0, P.stream>>>(y, a, x, b, 2 * n_complex);
}

}  // namespace akra
