// Legendre stages of the operator chain (device code, gfx950): the on-the-fly recurrences with
// exponent rescaling, the synthesis kernels (alm -> F per ring pair) and the adjoint kernels
// (G -> partial sums per ring block), plus the launch helpers shared by the translation units that
// instantiate them.  Not part of the public ABI.
//
// Two forms.  With W = (2lambda + -2lambda) / 2 and X = (2lambda - -2lambda) / 2, and the scalar functions
// l_lm = sqrt((2l+1)/4pi) d^l_{m0}(theta),
//   sin^2(theta) W_lm = w_2 l_{l+2} + w_0 l_l + w_-2 l_{l-2},   sin^2(theta) X_lm = x_1 l_{l+1} + x_-1 l_{l-1}
// with coefficients that depend on (l, m) only (see akra_internal.h).  So sin^2(theta) gamma_1 and
// sin^2(theta) gamma_2 are synthesised from scalar functions of degrees m .. lmax + 2, whose
// coefficients the prologue forms by a five-point stencil in l, and the adjoint is the transpose.
//   FORM_SCALAR, rings away from the poles: one recurrence of two instructions per degree (no b term)
//   and four multiply-adds serve both rings of a pair, against two recurrences of two FMAs each and
//   eight (one ring: four) multiply-adds in the spin form.
//   FORM_SPIN, the 64-pair groups that begin within AKRA_POLE_THETA or AKRA_POLE_X / lmax of a pole: there the
//   terms of the scalar sums cancel to sin^2(theta) of their size, and the spin-weighted functions themselves are run.
// Both are bounded by FP64 vector issue: the operands of a step are registers and one record, which
// the scalar synthesis reads from the lanes of a vector register and the others by scalar loads.  Every plan runs them in FP64: a plain FP32 FMA issues at the FP64 rate on this part
// (akra_fma_rate: 72 and 76 TFLOP/s), and an FP32 recurrence needs its coordinate as two floats, so
// FP32 arithmetic here costs more instructions for less precision.  FP32 plans store F, G and the
// partial sums as floats.
#pragma once
#include <type_traits>

#include "akra_fft.h"
#include "akra_internal.h"

namespace akra {
enum { FORM_SCALAR = 0, FORM_SPIN = 1 };
// ------------------------------------------------------------------------------------------------
// Entry states: stored in FP64 as mant * 2^(512 k).
// ------------------------------------------------------------------------------------------------
// spin form: i0, i1 = 1 / c_l and 1 / c_{l-1} at the entry degree l (mu = lambda / c).  refl = +-1
// gives the state of the reflected ring (theta -> pi - theta) instead: with s = refl = (-1)^(l+m) at
// the entry degree l, +2lambda_l(pi - theta) = s -2lambda_l(theta) and
// +2lambda_{l-1}(pi - theta) = -s -2lambda_{l-1}(theta), and the same with the spins exchanged.
__device__ __forceinline__ void load_entry_spin(const Ent64 *__restrict__ ent, const int *__restrict__ entk,
                                                int64_t idx, double i0, double i1, int refl, double &c2, double &p2,
                                                double &cm, double &pm, int &k)
{
    const Ent64 e = ent[idx];
    k = entk[idx];
    c2 = i0 * (refl ? refl * e.cm : e.c2);
    cm = i0 * (refl ? refl * e.c2 : e.cm);
    p2 = i1 * (refl ? -refl * e.pm : e.p2);
    pm = i1 * (refl ? -refl * e.p2 : e.pm);
}
// scalar form: the state is stored as mu; l_l(pi - theta) = s l_l(theta), l_{l-1}(pi - theta) = -s l_{l-1}(theta)
__device__ __forceinline__ void load_entry_scalar(const Ent64 *__restrict__ ent, const int *__restrict__ entk,
                                                  int64_t idx, int refl, double &c, double &p, int &k)
{
    const Ent64 e = ent[idx];
    k = entk[idx];
    c = refl ? refl * e.c2 : e.c2;
    p = refl ? -refl * e.p2 : e.p2;
}
// the batched FP32 kernels' near-polar groups: a spin entry state in their own unit, p2 and pm carrying
// lambda_l - lambda_{l-1} (the difference form)
__device__ __forceinline__ void load_entry_b(const Ent64 *__restrict__ ent, const int *__restrict__ entk, int64_t idx,
                                             float &c2, float &p2, float &cm, float &pm, int &k)
{
    const Ent64 e = ent[idx];
    const int k64 = entk[idx];
    const double d2 = e.c2 - e.p2, dm = e.cm - e.pm;
    const double big = fmax(fmax(fabs(e.c2), fabs(e.cm)), fmax(fabs(d2), fabs(dm)));
    if (big == 0.0) {
        c2 = p2 = cm = pm = 0.0f;
        k = 0;
        return;
    }
    const int ex = ilogb(big) + 512 * k64;
    const int k32 = (ex >= -40) ? 0 : -((20 - ex) / 64);
    const int sh = 512 * k64 - 64 * k32;
    c2 = (float)ldexp(e.c2, sh);
    p2 = (float)ldexp(d2, sh);
    cm = (float)ldexp(e.cm, sh);
    pm = (float)ldexp(dm, sh);
    k = k32;
}

template <typename T> __device__ __forceinline__ T scale_hi();
template <> __device__ __forceinline__ double scale_hi<double>() { return 0x1p256; }
template <> __device__ __forceinline__ float scale_hi<float>() { return 0x1p32f; }
template <typename T> __device__ __forceinline__ T scale_down();
template <> __device__ __forceinline__ double scale_down<double>() { return 0x1p-512; }
template <> __device__ __forceinline__ float scale_down<float>() { return 0x1p-64f; }

// A read-only pointer that is the same in every lane, made explicit for the compiler: the value is
// taken from the first lane and the result lives in the constant address space, so uniform loads
// through it become scalar loads.
template <typename P> using const_as = const __attribute__((address_space(4))) P;
template <typename P> __device__ __forceinline__ const_as<P> *uniform_ptr(const P *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const_as<P> *)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ Coef32D ld_coef(const_as<Coef32D> *p)
{
    Coef32D c;
    c.a = p->a;
    c.ep = p->ep;
    c.em = p->em;
    c.g = p->g;
    return c;
}

// The ring pair's position as the difference form uses it: y = 1 - cos(theta) (exact in double for the
// ring's defining z) as an unevaluated sum hi + lo of two floats.  Rounding it to one float would move
// the ring by a fixed angle, an error that grows linearly along l.
struct YF {
    float hi, lo;
};
__device__ __forceinline__ void setpos(YF &y, double z)
{
    const double v = 1.0 - z;
    y.hi = (float)v;
    y.lo = (float)(v - (double)y.hi);
}
// One step l -> l+1 of the spin +2 and spin -2 recurrences in the difference form: (c2, p2) = (lambda_l,
// lambda_l - lambda_{l-1}).
__device__ __forceinline__ void rstep(const Coef32D &c, YF y, float &c2, float &p2, float &cm, float &pm)
{
    const float t = c.a * y.lo;
    const float kp = fmaf(-c.a, y.hi, c.ep - t), km = fmaf(-c.a, y.hi, c.em - t);
    p2 = fmaf(kp, c2, c.g * p2);
    pm = fmaf(km, cm, c.g * pm);
    c2 += p2;
    cm += pm;
}

// One step of the scaled spin form (Coef64S): mu_{l+1} = (a' x +- b') mu_l - mu_{l-1}, two FMAs per spin.
__device__ __forceinline__ void rstep_s(double a, double b, double x, double &c2, double &p2, double &cm, double &pm)
{
    const double n2 = fma(fma(a, x, b), c2, -p2);
    const double nm = fma(fma(a, x, -b), cm, -pm);
    p2 = c2;
    c2 = n2;
    pm = cm;
    cm = nm;
}
// One step of the scaled scalar form: mu_{l+1} = a' x mu_l - mu_{l-1}.
__device__ __forceinline__ void rstep_0(double a, double x, double &c, double &p)
{
    const double n = fma(a * x, c, -p);
    p = c;
    c = n;
}

// wave-uniform "any lane"
__device__ __forceinline__ bool wave_any(bool p) { return __ballot(p) != 0ull; }

// first alm index of order m (the entry of l is base + l), and the same over the degrees m .. lmax + 2
// of the scalar functions (EXT_L more than lmax)
__device__ __forceinline__ int64_t alm_base(int m, int lmax) { return (int64_t)m * (2 * lmax + 1 - m) / 2; }
__device__ __forceinline__ int64_t ext_base(int m, int lmax) { return alm_base(m, lmax) + (int64_t)EXT_L * m; }

// The scalar form's coefficients q = (Re q_l, Im q_l, Re u_l, Im u_l) of entry (l, m), i its alm index (past
// the stored ones when l > lmax), of E, B = K_l (x_E, x_B) with Im(a_l0) dropped:
//   q_l = w_2(l-2) E_{l-2} + w_0(l) E_l + w_-2(l+2) E_{l+2} + i (x_1(l-1) B_{l-1} + x_-1(l+1) B_{l+1}),
//   u_l = w_2(l-2) B_{l-2} + w_0(l) B_l + w_-2(l+2) B_{l+2} - i (x_1(l-1) E_{l-1} + x_-1(l+1) E_{l+1})
// (the stencil is zero at degrees below 2, whose coefficients take no part whatever they hold).  All loads
// go out together, none behind a condition: a neighbour outside its column reads the entry nearest to it and counts as
// zero.  One neighbour after the other, the prologue waited for five latencies in turn (Nside 40: 5.3 us, so 4.0).
// K, E, B: kernel and coefficients of the entry itself, as they are stored.
__device__ __forceinline__ void stencil_in(const double2 *__restrict__ xE, const double2 *__restrict__ xB,
                                           const double *__restrict__ kern, const double *__restrict__ sten, int l,
                                           int m, int lmax, int64_t nalm, int64_t i, double (&q)[4], double &K,
                                           double2 &E, double2 &B)
{
    constexpr int row[5] = {ST_W2, ST_X1, ST_W0, ST_XM1, ST_WM2};  // of the neighbours l - 2 .. l + 2
    const int64_t ns = nalm + ALM_PAD;
    double w[5], k[5];
    double2 e[5], b[5];
#pragma unroll
    for (int n = 0; n < 5; ++n) {
        const int ln = l + n - 2, lc = ln < m ? m : ln > lmax ? lmax : ln;
        const int64_t ic = i - l + lc;
        w[n] = sten[row[n] * ns + ic];
        k[n] = kern ? kern[lc] : 1.0;
        e[n] = xE[ic];
        b[n] = xB[ic];
    }
    K = k[2];
    E = e[2];
    B = b[2];
    q[0] = q[1] = q[2] = q[3] = 0.0;
#pragma unroll
    for (int n = 0; n < 5; ++n) {
        const int ln = l + n - 2;
        const bool on = ln >= m && ln >= 2 && ln <= lmax;
        const double x = on ? w[n] * k[n] : 0.0;
        const double eR = on ? e[n].x : 0.0, eI = on && m ? e[n].y : 0.0;
        const double bR = on ? b[n].x : 0.0, bI = on && m ? b[n].y : 0.0;
        if (n & 1) {
            q[0] = fma(-x, bI, q[0]);
            q[1] = fma(x, bR, q[1]);
            q[2] = fma(x, eI, q[2]);
            q[3] = fma(-x, eR, q[3]);
        } else {
            q[0] = fma(x, eR, q[0]);
            q[1] = fma(x, eI, q[1]);
            q[2] = fma(x, bR, q[2]);
            q[3] = fma(x, bI, q[3]);
        }
    }
}

// XCD-aware placement: workgroups are dealt to the 8 XCDs round-robin, so all blocks of one m
// are mapped to blocks with the same index mod 8 (they share that XCD's L2 for the per-m data),
// and each XCD walks its m values in increasing order (decreasing work).  XCD x takes the orders
// m = 32 j + 4 x + i (i < 4): the four orders whose (Q, U) entries of one ring share a 128-byte
// line of F or G are placed on the same XCD, so the line is fetched into one L2, not four.  A
// launch covers m < 32 ceil((lmax + 1) / 32) (xcd_slots below); blocks past lmax return at once.
__device__ __forceinline__ void xcd_map(int b, int nbm, int &m, int &blk)
{
    const int xcd = b & 7, local = b >> 3;
    const int q = local / nbm;
    m = 32 * (q >> 2) + 4 * xcd + (q & 3);
    blk = local - q * nbm;
}

// Classes of 64-pair groups by the rings that carry weight (GCLS_BOTH, GCLS_NORTH, GCLS_SOUTH in
// akra_internal.h).  A one-ring class runs the recurrence on that ring itself (the south ring at its
// own cos(theta), from reflected entry states).

// Rescale of lane slot j once its values pass the upper bound; returns whether it left the scaled range.
template <int FORM>
__device__ __forceinline__ bool rescale_slot(double &c, double &p, double &cm, double &pm, int &k)
{
    const double big = FORM == FORM_SPIN ? fmax(fabs(c), fabs(cm)) : fabs(c);
    if (big <= scale_hi<double>()) return false;
    const double d = scale_down<double>();
    c *= d;
    p *= d;
    if (FORM == FORM_SPIN) {
        cm *= d;
        pm *= d;
    }
    k += 1;
    return k == 0;
}

template <int R> __device__ __forceinline__ bool pending(int l, int lmax, const int (&e)[R])
{
    bool q = false;
#pragma unroll
    for (int j = 0; j < R; ++j) q |= (e[j] > l && e[j] <= lmax);
    return q;
}

// ================================================================================================
// Legendre synthesis, scalar form.  For every (m, ring pair) the sums over l = m .. lmax + 2
//   S_q = sum q_l l_lm,  S_u = sum u_l l_lm            (q, u complex: the prologue's records)
// give sin^2(theta) (gamma_1, gamma_2) = -(S_q, S_u), so on the ring
//   F(m) = -(S_q + i S_u) / sin^2,   F(-m) = -(conj S_q + i conj S_u) / sin^2.
// The south ring of a pair takes the terms of odd l + m with the other sign: a two-sided class keeps
// the sums of even and odd l + m apart, a one-sided class sums all in one.  One wave handles the 64 R
// ring pairs of R list entries of one m: lane = pair, slot j = glist[w R + j] of wave w.  The records are the
// same for all lanes: lane n of every row of 16 loads that of degree l + n, 16 degrees ahead, and the FMAs
// take theirs from lane n of the row (a DPP operand, which costs no issue slot).  As scalar loads, whose
// wait covers all of them in flight, they could lead by two degrees only, and a wave waited for memory 64 to
// 73 % of its time where few waves share a SIMD.  Signs: with s = (+ + - -) over (l - m) mod 4, c and p hold s_l mu_l
// and s_{l-1} mu_{l-1}, and the records carry s_l and s_l s_{l+1}, so the recurrence is an accumulation,
//   p <- p + a (x c), then c and p change places.
// Bound by vector issue, six instructions per pair and degree: over all rings 5.6 ms at Nside 2048, lmax 4096,
// 0.80 of the FMA rate (5.6 with scalar loads, 11.1 in the spin form); Nside 512, lmax 1024 0.133 ms (0.141;
// 0.22), one ring of each pair 0.151 (0.198); northern footprint 75 || 57 us (115 || 109); Nside 256 0.054 (0.060).
// ================================================================================================
struct SRec {
    double a, q0, q1, u0, u1;  // a' of the scaled recurrence, c_l times Re q, Im q, Re u, Im u
};

// acc += r[lane N of the row] * c: the DPP operand of the FMA broadcasts within each row of 16 lanes
template <int N> __device__ __forceinline__ void fma_row(double &acc, double r, double c)
{
    asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(acc) : "v"(r), "v"(c), "n"(N));
}
// the same with the wait states (see settle) in front
template <int N> __device__ __forceinline__ void fma_row_settled(double &acc, double r, double c)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
        : "+v"(acc)
        : "v"(r), "v"(c), "n"(N));
}
// r's last write to its registers is two wait states back (a DPP operand's hazard after a vector write, which the
// compiler does not see in inline asm).  Due at the start of every straight run of fma_row: a register copy or
// reload may end the block before.
__device__ __forceinline__ void settle(SRec &r)
{
    asm volatile("s_nop 1" : "+v"(r.a), "+v"(r.q0), "+v"(r.q1), "+v"(r.u0), "+v"(r.u1));
}

// degree l + N of R pairs, r the records of l .. l + 15 in the lanes of each row
template <int N, int R>
__device__ __forceinline__ void syn_step(const SRec &r, const double (&x)[R], double (&c)[R], double (&p)[R],
                                         double (&acc)[4][R])
{
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const double t = x[j] * c[j];
        fma_row<N>(acc[0][j], r.q0, c[j]);
        fma_row<N>(acc[1][j], r.q1, c[j]);
        fma_row<N>(acc[2][j], r.u0, c[j]);
        fma_row<N>(acc[3][j], r.u1, c[j]);
        fma_row<N>(p[j], r.a, t);
        const double n = p[j];
        p[j] = c[j];
        c[j] = n;
    }
}
// the eight degrees l + N .. l + N + 7
template <int N, int R>
__device__ __forceinline__ void syn_steps8(const SRec &r, const double (&x)[R], double (&c)[R], double (&p)[R],
                                           double (&accA)[4][R], double (&accB)[4][R])
{
    syn_step<N, R>(r, x, c, p, accA);
    syn_step<N + 1, R>(r, x, c, p, accB);
    syn_step<N + 2, R>(r, x, c, p, accA);
    syn_step<N + 3, R>(r, x, c, p, accB);
    syn_step<N + 4, R>(r, x, c, p, accA);
    syn_step<N + 5, R>(r, x, c, p, accB);
    syn_step<N + 6, R>(r, x, c, p, accA);
    syn_step<N + 7, R>(r, x, c, p, accB);
}

template <typename S> __device__ __forceinline__ void syn_store(cplx<S> *f, double s0, double s1, double s2, double s3)
{
    f[0] = mk<S>((S)(s3 - s0), (S)(-(s1 + s2)));
    f[1] = mk<S>((S)(-(s0 + s3)), (S)(s1 - s2));
}

template <typename S, int R, int CLS>
__device__ __forceinline__ void syn_body(const double *__restrict__ recs, int64_t rec_stride, cplx<S> *__restrict__ FG,
                                         int64_t fg_stride, const Ent64 *__restrict__ ent,
                                         const int *__restrict__ entk, const int *__restrict__ entl, int ng64,
                                         const double *__restrict__ pair_z, int lmax, int npairs, int nrings,
                                         const int *__restrict__ glist, int ngl, int rhs, int m, int li0)
{
    const int lane = threadIdx.x & 63;
    constexpr bool TWO = CLS == GCLS_BOTH, REFL = CLS == GCLS_SOUTH;
    const int lend = lmax + EXT_L;
    const double *rec = recs + (rhs * rec_stride + ext_base(m, lmax)) * 5;

    double x[R], c[R], p[R], z2[R];
    int k[R], pr[R], e[R];
    double acc0[4][R], acc1[4][R];
    // entry degree of each slot's 64-pair group; the wave starts at the earliest
    const_as<int> *el = uniform_ptr(entl + (int64_t)m * ng64);
    const_as<int> *gl = uniform_ptr(glist);
    int ls = ENT_SKIP;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int g = li0 + j < ngl ? gl[li0 + j] : -1;
        e[j] = g >= 0 ? el[g] : ENT_SKIP;
        ls = e[j] < ls ? e[j] : ls;
        pr[j] = g >= 0 ? g * 64 + lane : npairs;  // pairs at or past npairs hold nothing
    }
    const int64_t row = (int64_t)m * npairs;
    // start of the slots whose group enters at l (their values are zero until then)
    auto enter = [&](int l) {
        const int refl = REFL ? (((l + m) & 1) ? -1 : 1) : 0;
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (e[j] == l && pr[j] < npairs) {
                load_entry_scalar(ent, entk, row + pr[j], refl, c[j], p[j], k[j]);
                p[j] = -p[j];
            }
    };
    auto scaled = [&]() {
        bool neg = false;
#pragma unroll
        for (int j = 0; j < R; ++j) neg |= (k[j] < 0);
        return wave_any(neg);
    };
#pragma unroll
    for (int j = 0; j < R; ++j) {
        x[j] = c[j] = p[j] = 0.0;
        k[j] = 0;
        if (pr[j] < npairs) x[j] = REFL ? -pair_z[pr[j]] : pair_z[pr[j]];
        z2[j] = x[j];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc0[q][j] = acc1[q][j] = 0.0;
    }
    if (ls <= lend) enter(ls);
    // Lanes whose scale exponent is still negative ("ramp") run the same unmasked steps: their
    // scaled values accumulate garbage that is discarded when the lane's exponent reaches zero (its
    // sums restart there) or at the end; the check runs once per eight steps, which the growth
    // of the recurrence keeps far from overflow.
    bool pend = R > 1 && pending<R>(ls, lend, e);
    bool ramp = scaled();
    // entries are m + 8 q, so l + m is even at the start of every eight degrees
    double(&accB)[4][R] = TWO ? acc1 : acc0;
    auto load = [&](int l) {
        const int i = l + (lane & 15);
        const double *r = rec + (int64_t)5 * (i < lend ? i : lend);
        SRec s;
        s.a = r[0];
        s.q0 = r[1];
        s.q1 = r[2];
        s.u0 = r[3];
        s.u1 = r[4];
        return s;
    };
    auto before = [&](int l) {
        if (!pend) return;
        enter(l);
        pend = pending<R>(l, lend, e);
        ramp = ramp || scaled();
    };
    auto after = [&]() {
        if (!ramp) return;
        bool neg = false;
        double no = 0.0;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (k[j] < 0 && rescale_slot<FORM_SCALAR>(c[j], p[j], no, no, k[j])) {
#pragma unroll
                for (int q = 0; q < 4; ++q) acc0[q][j] = acc1[q][j] = 0.0;
            }
            neg |= (k[j] < 0);
        }
        ramp = wave_any(neg);
    };
    int l = __builtin_amdgcn_readfirstlane(ls <= lend ? ls : lend + 1);
    SRec r = load(l);
    for (; l <= lend; l += 16) {
        if (l + 15 > lend && l + (lane & 15) > lend) r.a = r.q0 = r.q1 = r.u0 = r.u1 = 0.0;
        SRec n = load(l + 16);
        before(l);
        settle(r);
        syn_steps8<0, R>(r, x, c, p, acc0, accB);
        after();
        if (l + 8 > lend) break;
        before(l + 8);
        settle(r);
        syn_steps8<8, R>(r, x, c, p, acc0, accB);
        after();
        r = n;
    }
    cplx<S> *Fb = FG + rhs * fg_stride;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if (pr[j] >= npairs) continue;
        // lanes that never left the scaled range contribute nothing
        const double f = k[j] < 0 ? 0.0 : 1.0 / ((1.0 - z2[j]) * (1.0 + z2[j]));
        double s[4], t[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double E = k[j] < 0 ? 0.0 : acc0[q][j], O = k[j] < 0 ? 0.0 : acc1[q][j];
            s[q] = f * (E + O);
            t[q] = f * (E - O);
        }
        const int rn = pr[j], rs = nrings - 1 - pr[j];
        if (CLS != GCLS_SOUTH)
            syn_store<S>(Fb + ((int64_t)rn * (lmax + 1) + m) * 2, s[0], s[1], s[2], s[3]);
        // (the equator ring belongs to the north side)
        if (CLS == GCLS_SOUTH && rs != rn)
            syn_store<S>(Fb + ((int64_t)rs * (lmax + 1) + m) * 2, s[0], s[1], s[2], s[3]);
        if (TWO && rs != rn) syn_store<S>(Fb + ((int64_t)rs * (lmax + 1) + m) * 2, t[0], t[1], t[2], t[3]);
    }
}

// ================================================================================================
// Legendre synthesis, spin form: one wave per (m, near-polar 64-pair group), sums over l = max(m,2) ..
// lmax of the spin +2 and -2 values times the records in the u basis
//   u0 = aE.re - aB.im,  u1 = aE.im + aB.re,  u2 = aE.re + aB.im,  u3 = aB.re - aE.im.
// S+(u) and S-(u) being the sums of the spin +-2 values times u, the north ring takes
//   F(m) = -(S+(u0), S+(u1)),  F(-m) = -(S-(u2), S-(u3)),
// and the south ring, by 2lambda_lm(pi - theta) = (-1)^(l+m) -2lambda_lm(theta), S-(u0), S-(u1), S+(u2),
// S+(u3) with the sign of l + m.
// ================================================================================================
struct SpinRec {
    double a, b, u0, u1, u2, u3;  // a', b' of the scaled form; c_l times the u combinations
};
static_assert(sizeof(SpinRec) == SPIN_REC * sizeof(double), "allocation of the records");

template <typename S, int CLS>
__device__ __forceinline__ void spin_body(const SpinRec *__restrict__ recs, int64_t rec_stride,
                                          const Coef64S *__restrict__ cs64, cplx<S> *__restrict__ FG,
                                          int64_t fg_stride, const Ent64 *__restrict__ ent,
                                          const int *__restrict__ entk, const int *__restrict__ entl, int ng64,
                                          const double *__restrict__ pair_z, int lmax, int npairs, int nrings, int g,
                                          int rhs, int m)
{
    const int lane = threadIdx.x & 63;
    constexpr bool TWO = CLS == GCLS_BOTH, REFL = CLS == GCLS_SOUTH;
    const int l0 = m > 2 ? m : 2;
    const int64_t base = alm_base(m, lmax);
    const_as<Coef64S> *ct = uniform_ptr(cs64 + base);
    const int ls = uniform_ptr(entl + (int64_t)m * ng64)[g];
    const int pr = g * 64 + lane;
    double x = 0, c2 = 0, p2 = 0, cm = 0, pm = 0;
    int k = 0;
    if (pr < npairs && ls <= lmax) {
        x = REFL ? -pair_z[pr] : pair_z[pr];
        load_entry_spin(ent, entk, (int64_t)m * npairs + pr, ct[ls].ic, ct[ls - 1].ic,
                        REFL ? (((ls + m) & 1) ? -1 : 1) : 0, c2, p2, cm, pm, k);
    }
    // a[0..3] of the even steps from ls, b of the odd ones: S+(u0), S+(u1), S-(u2), S-(u3) and, for the
    // south ring of a two-sided group, S-(u0), S-(u1), S+(u2), S+(u3)
    double a[8], b[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q] = b[q] = 0.0;
    const_as<SpinRec> *rp = uniform_ptr(recs + rhs * rec_stride + base);
    auto ld = [&](int i) {
        SpinRec r;
        r.a = rp[i].a;
        r.b = rp[i].b;
        r.u0 = rp[i].u0;
        r.u1 = rp[i].u1;
        r.u2 = rp[i].u2;
        r.u3 = rp[i].u3;
        return r;
    };
    auto step = [&](const SpinRec &in, double (&s)[8]) {
        s[0] = fma(c2, in.u0, s[0]);
        s[1] = fma(c2, in.u1, s[1]);
        s[2] = fma(cm, in.u2, s[2]);
        s[3] = fma(cm, in.u3, s[3]);
        if (TWO) {
            s[4] = fma(cm, in.u0, s[4]);
            s[5] = fma(cm, in.u1, s[5]);
            s[6] = fma(c2, in.u2, s[6]);
            s[7] = fma(c2, in.u3, s[7]);
        }
        rstep_s(in.a, in.b, x, c2, p2, cm, pm);
    };
    bool ramp = wave_any(k < 0);
    int l = __builtin_amdgcn_readfirstlane(ls <= lmax ? ls : lmax + 1);
    // four degrees per trip, their records loaded a trip ahead: the few waves of these groups have
    // little beside them to hide a load's latency (the record buffer is padded)
    SpinRec r[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) r[t] = ld(l + t);
    for (; l + 3 <= lmax; l += 4) {
        SpinRec n[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) n[t] = ld(l + 4 + t);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (t & 1) step(r[t], b);
            else step(r[t], a);
        }
        if (ramp) {
            // the sums of a lane that leaves the scaled range restart there
            if (k < 0 && rescale_slot<FORM_SPIN>(c2, p2, cm, pm, k)) {
#pragma unroll
                for (int q = 0; q < 8; ++q) a[q] = b[q] = 0.0;
            }
            ramp = wave_any(k < 0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) r[t] = n[t];
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        if (l + t > lmax) break;
        if (t & 1) step(r[t], b);
        else step(r[t], a);
    }
    if (pr >= npairs) return;
    const bool odd0 = ((l0 + m) & 1) != 0;  // entries are l0 + 8 q: a holds l + m odd when true
    cplx<S> *Fb = FG + rhs * fg_stride;
    const int rn = pr, rs = nrings - 1 - pr;
    double s[8];  // lanes that never left the scaled range contribute nothing
#pragma unroll
    for (int q = 0; q < 8; ++q) s[q] = k < 0 ? 0.0 : q < 4 ? a[q] + b[q] : odd0 ? b[q] - a[q] : a[q] - b[q];
    if (CLS != GCLS_SOUTH || rs != rn) {
        cplx<S> *f = Fb + ((int64_t)(CLS == GCLS_SOUTH ? rs : rn) * (lmax + 1) + m) * 2;
        f[0] = mk<S>((S)-s[0], (S)-s[1]);
        f[1] = mk<S>((S)-s[2], (S)-s[3]);
    }
    if (TWO && rs != rn) {
        cplx<S> *f = Fb + ((int64_t)rs * (lmax + 1) + m) * 2;
        f[0] = mk<S>((S)-s[4], (S)-s[5]);
        f[1] = mk<S>((S)-s[6], (S)-s[7]);
    }
}

// Synthesis over a list of 64-pair groups: the first nspin waves of an m run one spin group each, the
// others R of the ngl scalar groups that follow; four waves per workgroup, nbm workgroups per m.
template <typename S, int R, int CLS>
__global__ __launch_bounds__(256) void k_leg_synth(const double *__restrict__ recs, int64_t rec_stride,
                                                   const SpinRec *__restrict__ srecs, int64_t srec_stride,
                                                   const Coef64S *__restrict__ cs64, cplx<S> *__restrict__ FG,
                                                   int64_t fg_stride, const Ent64 *__restrict__ ent,
                                                   const int *__restrict__ entk, const int *__restrict__ entl,
                                                   int ng64, const double *__restrict__ pair_z, int lmax, int npairs,
                                                   int nrings, const int *__restrict__ glist, int nspin, int ngl,
                                                   int nbm)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int m, blk;
    xcd_map((int)blockIdx.x, nbm, m, blk);
    const int w = blk * 4 + wave, li0 = (w - nspin) * R;
    if (m > lmax || li0 >= ngl) return;
    if (w < nspin) {
        spin_body<S, CLS>(srecs, srec_stride, cs64, FG, fg_stride, ent, entk, entl, ng64, pair_z, lmax, npairs, nrings,
                          uniform_ptr(glist)[w], blockIdx.y, m);
        return;
    }
    syn_body<S, R, CLS>(recs, rec_stride, FG, fg_stride, ent, entk, entl, ng64, pair_z, lmax, npairs, nrings,
                        glist + nspin, ngl, blockIdx.y, m, li0);
}

// ================================================================================================
// Legendre adjoint: for one m and a block of ring pairs, the partial sums over the block's rings
//   scalar form  T_1 = sum_r l_lm(theta_r) g_1(m) / sin^2(theta_r),  T_2 the same with g_2, where
//                g_1 = (G(m) + conj G(-m)) / 2 and g_2 = (G(m) - conj G(-m)) / 2i are the ring's Fourier
//                coefficients of the two weighted shear components; l = m .. lmax + 2, in units of mu
//                (the epilogue multiplies by c_l and applies the transposed stencil)
//   spin form    2h = sum_r 2lambda_lm(theta_r) G_r(m),  -2h = sum_r -2lambda_lm(theta_r) conj(G_r(-m))
// (south rings through the reflection symmetry).  Each lane sums its R ring pairs in registers; each
// degree's four sums are added over the four rows of the wave in registers (row_sum4: six lane swaps and
// three adds), and every L steps of l the sixteen partials per output and wave go through LDS; a single-wave workgroup sums
// them during the next L steps (waiting for them at once: 0.097 ms against 0.087 at Nside 256, lmax 512, and
// 5 % of a 512 mixed solve).  With
// every lane's partials through LDS instead (four writes and four reads per degree), the LDS time of a
// degree was that of five to six ring pairs' FMAs and did not hide behind them.  Adjoint and epilogue
// over all rings: Nside 2048, lmax 4096, 4 pairs per lane 10.7 -> 9.2 ms, 8 pairs 8.5 -> 7.9 ms (spin
// form before: 13.8 ms); Nside 512, lmax 1024, 4 pairs 0.40 -> 0.25 ms.  What bounds it now is vector issue:
// six instructions per pair and eleven for the reduction per degree, at 0.72 of the FMA rate.
// ga, gb: the values a slot contracts with.  Scalar form: a two-sided class holds north + south for
// even l + m and north - south for odd, a one-sided class its ring's in ga.  Spin form: ga = (G_N,
// conj H_N), gb = the south ring's.
// ================================================================================================
template <int FORM, int R, bool ODD, int CLS>
__device__ __forceinline__ void adj_step(double ca, double cb, const double (&x)[R], double (&c)[R], double (&p)[R],
                                         double (&cm)[R], double (&pm)[R], const double (&ga)[4][R],
                                         const double (&gb)[4][R], double (&out)[4])
{
    double o[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < R; ++j) {
        if constexpr (FORM == FORM_SCALAR) {
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = fma(c[j], (ODD && CLS == GCLS_BOTH) ? gb[q][j] : ga[q][j], o[q]);
            rstep_0(ca, x[j], c[j], p[j]);
        } else {
            const double s = ODD ? -1.0 : 1.0;
            if (CLS != GCLS_SOUTH) {
                o[0] = fma(c[j], ga[0][j], o[0]);
                o[1] = fma(c[j], ga[1][j], o[1]);
                o[2] = fma(cm[j], ga[2][j], o[2]);
                o[3] = fma(cm[j], ga[3][j], o[3]);
            }
            if (CLS != GCLS_NORTH) {
                o[0] = fma(s * cm[j], gb[0][j], o[0]);
                o[1] = fma(s * cm[j], gb[1][j], o[1]);
                o[2] = fma(s * c[j], gb[2][j], o[2]);
                o[3] = fma(s * c[j], gb[3][j], o[3]);
            }
            rstep_s(ca, cb, x[j], c[j], p[j], cm[j], pm[j]);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) out[q] = o[q];
}

// Occupancy the adjoint is compiled for (waves per SIMD).  A slot of the scalar form holds x, mu_l,
// mu_{l-1} and four (one-sided) or eight values of G.  Six two-sided slots do not fit in the 168 registers of
// three waves (202 spilled, 17 reloads per eight degrees; two waves: 7 spilled): all rings, two / three waves, FP64 and
// FP32, ms, lmax 4096 7.80 / 8.27 and 7.57 / 7.90, lmax 2048 1.00 / 1.16 and 0.96 / 1.06.  Five two-sided slots (76
// spilled) and eight one-sided (142) are as good or better with three: lmax 4096 8.12 / 7.75 and 7.29 / 6.96.
template <int R, int CLS> struct AdjWaves {
    static constexpr bool two = CLS == GCLS_BOTH;
    static constexpr int value = two ? (R <= 2 ? 4 : R <= 5 ? 3 : 2) : (R <= 4 ? 4 : R <= 8 ? 3 : 2);
};
// LDS hand-over between the lanes of a workgroup.  A single-wave workgroup needs no s_barrier: the
// LDS unit executes one wave's instructions in order, so a fence that keeps the compiler from moving
// LDS accesses across it suffices, and no full wait for outstanding LDS operations is forced.
// value of lane l ^ 1, l ^ 2 (DPP quad permutations) and of the mirrored lane in the half-row of
// 8 or the row of 16 lanes (row_half_mirror, row_mirror)
template <int CTRL> __device__ __forceinline__ float dpp_mov(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
// sum over the aligned group of G lanes (G = 1, 2, 4, 8, 16), in every lane of the group
template <int G, typename T> __device__ __forceinline__ T group_sum(T s)
{
    static_assert(G == 1 || G == 2 || G == 4 || G == 8 || G == 16, "group size");
    if constexpr (G >= 2) s += dpp_mov<0xB1>(s);   // quad_perm [1, 0, 3, 2]
    if constexpr (G >= 4) s += dpp_mov<0x4E>(s);   // quad_perm [2, 3, 0, 1]
    if constexpr (G >= 8) s += dpp_mov<0x141>(s);  // row_half_mirror: lane 7 - i of the half-row
    if constexpr (G >= 16) s += dpp_mov<0x140>(s); // row_mirror: lane 15 - i of the row
    return s;
}

// Exchange between the halves of a wave (rows of 16 lanes r0 r1 r2 r3): a = [a0 a1 b0 b1],
// b = [a2 a3 b2 b3]; and between its odd and even rows: a = [a0 b0 a2 b2], b = [a1 b1 a3 b3].
__device__ __forceinline__ void swap_halves(double &a, double &b)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(hi[0], lo[0]);
    b = __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ void swap_rows(double &a, double &b)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
    a = __hiloint2double(hi[0], lo[0]);
    b = __hiloint2double(hi[1], lo[1]);
}
// The four outputs of a degree summed over the four rows of the wave: lane (q, j) = (lane / 16, lane % 16)
// returns the sum of output q over the lanes j, j + 16, j + 32, j + 48.
__device__ __forceinline__ double row_sum4(double (&o)[4])
{
    swap_halves(o[0], o[2]);
    swap_halves(o[1], o[3]);
    double a = o[0] + o[2], b = o[1] + o[3];
    swap_rows(a, b);
    return a + b;
}

template <int W> __device__ __forceinline__ void wg_lds_sync()
{
    if constexpr (W == 1) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// The adjoint of one workgroup: m, its ring block rb, and its groups glist[lw .. lw + W R) (wave w
// the R of them from lw + w R; entries at or past ngl hold nothing).  red: the workgroup's LDS.
template <int FORM, typename S, int R, int W, int L, int CLS>
__device__ __forceinline__ void adj_body(double *__restrict__ red, const cplx<S> *__restrict__ FG,
                                         const double *__restrict__ sa, const Coef64S *__restrict__ cs64,
                                         const Ent64 *__restrict__ ent, const int *__restrict__ entk,
                                         const int *__restrict__ entl, int ng64, const double *__restrict__ pair_z,
                                         S *__restrict__ part, int *__restrict__ wgstart, int64_t slab, int lmax,
                                         int npairs, int nrings, const int *__restrict__ glist, int ngl,
                                         const uint8_t *__restrict__ live, int nrb, int m, int rb, int lw)
{
    // LDS rows (l) of W waves x 4 outputs x 16 partials, padded to CS entries: the G threads that sum
    // one output read its entries gi + G t, and with CS = 64 W + G (mod 32 double-banks) the 64 threads
    // of a wave spread over the banks twice each, as do the lane-contiguous writes
    constexpr int GR = 16 * W / L, CS = 64 * W + GR;
    constexpr bool SPIN = FORM == FORM_SPIN, REFL = !SPIN && CLS == GCLS_SOUTH;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int l0 = SPIN && m < 2 ? 2 : m, lend = SPIN ? lmax : lmax + EXT_L;
    const int64_t base = SPIN ? alm_base(m, lmax) : ext_base(m, lmax);
    const_as<Coef64S> *ct = uniform_ptr(SPIN ? cs64 + base : cs64);
    const double sgn0 = ((l0 + m) & 1) ? -1.0 : 1.0;

    // entry degrees of the workgroup's 64-pair groups: the workgroup starts at the earliest, a slot
    // whose group enters later holds zeros until its entry (always at a chunk start: entries are
    // l0 + 8q and chunks start at l0 + Lq)
    const_as<int> *el = uniform_ptr(entl + (int64_t)m * ng64);
    const_as<int> *gl = uniform_ptr(glist);
    int ls = ENT_SKIP;
    for (int li = lw; li < lw + W * R && li < ngl; ++li) ls = el[gl[li]] < ls ? el[gl[li]] : ls;
    if (threadIdx.x == 0) wgstart[(int64_t)m * nrb + rb] = ls;
    if (ls > lend) return;
    int e[R], gs[R];  // wave-uniform: entry degree and group of each slot (ng64: none)
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int li = lw + wave * R + j;
        const int g = li < ngl ? gl[li] : -1;
        e[j] = g >= 0 ? el[g] : ENT_SKIP;
        gs[j] = g >= 0 ? g : ng64;
    }
    const int64_t row = (int64_t)m * npairs;
    auto pr = [&](int j) { return gs[j] * 64 + lane; };  // pairs at or past npairs hold nothing

    double x[R], c[R], p[R], cm[R], pm[R], ga[4][R], gb[4][R];
    int k[R];
    // start of the slots whose group enters at l (their values are zero until then)
    auto enter = [&](int l) {
        const int refl = REFL ? (((l + m) & 1) ? -1 : 1) : 0;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (e[j] != l || pr(j) >= npairs) continue;
            if constexpr (SPIN)
                load_entry_spin(ent, entk, row + pr(j), ct[l].ic, ct[l - 1].ic, 0, c[j], p[j], cm[j], pm[j], k[j]);
            else
                load_entry_scalar(ent, entk, row + pr(j), refl, c[j], p[j], k[j]);
        }
    };
    // G of slot j's ring pair; lanes still in the scaled range (k < 0) hold G = 0, so the unmasked
    // steps add nothing for them until their exponent reaches zero and G is loaded
    auto load_g = [&](int j) {
        const int q = pr(j);
        if (q >= npairs || k[j] < 0) return;
        const int rn = q, rs = nrings - 1 - q;
        double n[4] = {0, 0, 0, 0}, s[4] = {0, 0, 0, 0};
        // Re, Im of G(m) and of conj G(-m)
        auto get = [&](int r, double (&v)[4]) {
            const cplx<S> *f = FG + ((int64_t)r * (lmax + 1) + m) * 2;
            const cplx<S> g = f[0], h = f[1];
            v[0] = g.x;
            v[1] = g.y;
            v[2] = h.x;
            v[3] = -(double)h.y;
        };
        if (CLS != GCLS_SOUTH && (!live || live[rn])) get(rn, n);
        if (CLS != GCLS_NORTH && rs != rn && (!live || live[rs])) get(rs, s);
        if constexpr (SPIN) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                ga[t][j] = n[t];
                gb[t][j] = sgn0 * s[t];
            }
        } else {
            // g_1 and g_2 over sin^2
            const double f = 0.5 / ((1.0 - x[j]) * (1.0 + x[j]));
            auto comp = [&](const double (&v)[4], double (&o)[4]) {
                o[0] = f * (v[0] + v[2]);
                o[1] = f * (v[1] + v[3]);
                o[2] = f * (v[1] - v[3]);
                o[3] = f * (v[2] - v[0]);
            };
            double a[4], b[4];
            comp(n, a);
            comp(s, b);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                ga[t][j] = a[t] + b[t];
                if (CLS == GCLS_BOTH) gb[t][j] = a[t] - b[t];
            }
        }
        // one slot after the other: the loads of all slots at once would set the kernel's register count
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int j = 0; j < R; ++j) {
        x[j] = c[j] = cm[j] = p[j] = pm[j] = 0.0;
        k[j] = 0;
        if (pr(j) < npairs) x[j] = REFL ? -pair_z[pr(j)] : pair_z[pr(j)];
#pragma unroll
        for (int t = 0; t < 4; ++t) ga[t][j] = gb[t][j] = 0.0;
    }
    enter(ls);
    bool neg = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        neg |= (k[j] < 0);
        if (e[j] == ls) load_g(j);
    }
    bool ramp = wave_any(neg);
    bool pend = (R > 1 || W > 1) && pending<R>(ls, lend, e);
    constexpr int NT = 64 * W, NO = 4 * L, G = NT / NO;
    static_assert(G == GR && G >= 1 && 16 % G == 0 && L >= 4, "reduction layout");
    const int t = threadIdx.x, o = t / G, gi = t - o * G;
    const int oli = o >> 2, oc = o & 3;
    const double *col = red + oli * CS + oc * 16 + gi;              // output o, entry gi
    double *rw = red + wave * 64 + lane;
    S *pout = part + ((int64_t)rb * slab + base + ls + oli) * 4 + oc;  // output of the first chunk

    // coefficients through an explicitly uniform pointer (scalar loads); the tables are padded past
    // their last column, so the look-ahead loads stay in bounds
    const_as<double> *sp = uniform_ptr(SPIN ? sa : sa + base + ls);
    const_as<Coef64S> *cp = SPIN ? ct + ls : ct;
    double cca[L], ccb[L];
    auto ldc = [&](int i, double &a, double &b) {
        a = SPIN ? cp[i].a : sp[i];
        b = SPIN ? cp[i].b : 0.0;
    };
#pragma unroll
    for (int li = 0; li < L; ++li) ldc(li, cca[li], ccb[li]);
    // sums over the 16 W partials of an output: thread (o, gi) reads the entries gi + G u of output o
    // (wave / 16, partial % 16) at compile-time offsets, adds them in four independent partial
    // sums, then sums over the G adjacent threads sharing the output with DPP lane moves
    double rv[L], sc = 1.0;
    auto read = [&]() {
#pragma unroll
        for (int u = 0; u < L; ++u) rv[u] = col[(G * u / 16) * 64 + (G * u) % 16];
    };
    auto finish = [&](int l, double c_l) {
        double ps[4];
#pragma unroll
        for (int u = 0; u < L; ++u) {
            if (u < 4) ps[u] = rv[u];
            else ps[u & 3] += rv[u];
        }
        const double s = group_sum<G>((ps[0] + ps[1]) + (ps[2] + ps[3]));
        if (gi == 0 && l >= ls && l + oli <= lend) pout[(int64_t)(l - ls) * 4] = (S)(SPIN ? s * c_l : s);
    };
#pragma unroll
    for (int u = 0; u < L; ++u) rv[u] = 0.0;
    for (int lc = ls; lc <= lend; lc += L, cp += SPIN ? L : 0, sp += SPIN ? 0 : L) {
        if (pend) {
            enter(lc);
            bool ng = false;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (e[j] == lc) load_g(j);
                ng |= (k[j] < 0);
            }
            ramp = ramp || wave_any(ng);
            pend = pending<R>(lc, lend, e);
        }
        // the next chunk's coefficients (scalar loads) are issued before this chunk's steps: they
        // share the LDS wait counter, and must have arrived by the time the reduction waits on LDS
        double nca[L], ncb[L];
#pragma unroll
        for (int li = 0; li < L; ++li) ldc(L + li, nca[li], ncb[li]);
        // c_l of this thread's output row in the spin form (a vector load, used at the store)
        const double scp = sc;
        if constexpr (SPIN) sc = cs64[base + (lc + oli < lmax ? lc + oli : lmax)].c;
        // all L steps unmasked: rows past lend (last chunk) are reduced but not stored, and the
        // coefficient table is padded past its last column
#pragma unroll
        for (int li = 0; li < L; li += 2) {
            // A single-wave workgroup reads a chunk's partials as soon as they are written and sums them
            // in the middle of the next chunk's steps (its LDS accesses execute in order, so the next
            // writes cannot pass the reads)
            if (W == 1 && li == L / 2) {
                __builtin_amdgcn_sched_barrier(0);
                finish(lc - L, scp);
                __builtin_amdgcn_sched_barrier(0);
            }
            double out[4];
            adj_step<FORM, R, false, CLS>(cca[li], ccb[li], x, c, p, cm, pm, ga, gb, out);
            rw[li * CS] = row_sum4(out);
            adj_step<FORM, R, true, CLS>(cca[li + 1], ccb[li + 1], x, c, p, cm, pm, ga, gb, out);
            rw[(li + 1) * CS] = row_sum4(out);
        }
        wg_lds_sync<W>();
        read();
        if (W > 1) finish(lc, sc);
#pragma unroll
        for (int li = 0; li < L; ++li) {
            cca[li] = nca[li];
            ccb[li] = ncb[li];
        }
        if (ramp) {
            // once per chunk (the growth over L steps stays far from overflow): rescale, and load
            // G for lanes whose exponent reached zero
            bool any_neg = false;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (k[j] < 0 && rescale_slot<FORM>(c[j], p[j], cm[j], pm[j], k[j])) load_g(j);
                any_neg |= (k[j] < 0);
            }
            ramp = wave_any(any_neg);
        }
        wg_lds_sync<W>();
    }
    if (W == 1) finish(ls + (lend - ls) / L * L, sc);
}

// Adjoint over a list of 64-pair groups, the first nspin of them (nearest the poles) in the spin form.
// Of the nbs + nbm workgroups of every m the first nbs take spin_gpb(W) spin groups each and write ring
// blocks rbs .., the others the ngl scalar groups that follow in the list as adj_block gives them (W R
// each for W > 1; for W = 1 the first nA workgroups R groups each and the others R - 1, so that no slot
// is empty) and write ring blocks rbm ...  One launch holds both forms, so the few long recurrences of the
// spin groups run beside the others.  CLS selects the rings it reads (GCLS_BOTH, GCLS_NORTH, GCLS_SOUTH);
// a ring whose flag in live is zero is read as G = 0 (live null: every ring is read).
template <typename S, int R, int W, int L, int CLS>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(AdjWaves<R, CLS>::value))) void k_leg_adj(
    const cplx<S> *__restrict__ FG, const double *__restrict__ sa, const Coef64S *__restrict__ cs64,
    const Ent64 *__restrict__ ent, const int *__restrict__ entk, const int *__restrict__ entl, int ng64,
    const double *__restrict__ pair_z, S *__restrict__ part, int *__restrict__ wgstart, int64_t slab, int lmax,
    int npairs, int nrings, const int *__restrict__ glist, int nspin, int ngl, const uint8_t *__restrict__ live,
    int rbs, int rbm, int nbs, int nbm, int nrb, int nA)
{
    __shared__ double red[L * (64 * W + 16 * W / L)];
    int m, b;
    xcd_map((int)blockIdx.x, nbs + nbm, m, b);
    if (m > lmax) return;
    if (b < nbs) {
        if constexpr (W == 1) {
            // a workgroup with one spin group left runs no empty slot
            if (b * spin_gpb(W) + 1 == nspin) {
                adj_body<FORM_SPIN, S, 1, W, L, CLS>(red, FG, sa, cs64, ent, entk, entl, ng64, pair_z, part, wgstart,
                                                     slab, lmax, npairs, nrings, glist, nspin, live, nrb, m, rbs + b,
                                                     b * spin_gpb(W));
                return;
            }
        }
        adj_body<FORM_SPIN, S, spin_gpb(W) / W, W, L, CLS>(red, FG, sa, cs64, ent, entk, entl, ng64, pair_z, part,
                                                               wgstart, slab, lmax, npairs, nrings, glist, nspin,
                                                               live, nrb, m, rbs + b, b * spin_gpb(W));
        return;
    }
    b -= nbs;
    if constexpr (W == 1 && R > 1) {
        if (b >= nA) {
            adj_body<FORM_SCALAR, S, R - 1, 1, L, CLS>(red, FG, sa, cs64, ent, entk, entl, ng64, pair_z, part, wgstart,
                                                       slab, lmax, npairs, nrings, glist + nspin, ngl, live, nrb, m,
                                                       rbm + b, nA * R + (b - nA) * (R - 1));
            return;
        }
    }
    adj_body<FORM_SCALAR, S, R, W, L, CLS>(red, FG, sa, cs64, ent, entk, entl, ng64, pair_z, part, wgstart, slab, lmax,
                                           npairs, nrings, glist + nspin, ngl, live, nrb, m, rbm + b, b * W * R);
}

// ================================================================================================
// launch helpers (host): the translation units akra_leg_both/north/south.hip instantiate
// leg_synth_cls and leg_adj_cls for one class each
// ================================================================================================
inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
// orders per XCD of a launch placed by xcd_map: 8 of them cover 32 ceil((lmax + 1) / 32) >= lmax + 1
inline int64_t xcd_slots(int lmax) { return 4 * cdiv(lmax + 1, 32); }

template <typename S, int R, int CLS>
void syn_launch(Plan &P, int nrhs, const int *list, int nspin, int nmain)
{
    const int64_t fg_stride = (int64_t)P.nrings * (P.lmax + 1) * 2;
    const int nbm = (int)cdiv(nspin + cdiv(nmain, R), 4);  // workgroups per m
    dim3 g((unsigned)(8 * nbm * xcd_slots(P.lmax)), nrhs);
    k_leg_synth<S, R, CLS><<<g, 256, 0, P.stream>>>(
        P.d_rec, P.rec_stride, (const SpinRec *)P.d_rec_spin, P.nalm + ALM_PAD, P.d_coef64s, (cplx<S> *)P.d_FG,
        fg_stride, P.d_ent, P.d_entk, P.d_entl, P.ng64, P.d_pair_z, P.lmax, P.npairs, P.nrings, list, nspin, nmain, nbm);
}

// launch shape of a class: the two-sided class takes (syn_R, adj_R, adj_W, adj_L), the
// one-sided classes (syn_R1, adj_R1, adj_W1, adj_L1)
inline int syn_R_of(const Plan &P, int cls) { return cls == GCLS_BOTH ? P.syn_R : P.syn_R1; }
inline void adj_shape_of(const Plan &P, int cls, int &R, int &W, int &L)
{
    R = cls == GCLS_BOTH ? P.adj_R : P.adj_R1;
    W = cls == GCLS_BOTH ? P.adj_W : P.adj_W1;
    L = cls == GCLS_BOTH ? P.adj_L : P.adj_L1;
}

template <typename S, int CLS>
void leg_synth_s(Plan &P, int nrhs, const int *list, int nspin, int nmain)
{
    const int R = syn_R_of(P, CLS);
    if (R == 1) syn_launch<S, 1, CLS>(P, nrhs, list, nspin, nmain);
    else if (R == 2) syn_launch<S, 2, CLS>(P, nrhs, list, nspin, nmain);
    else syn_launch<S, 4, CLS>(P, nrhs, list, nspin, nmain);
}

// Legendre synthesis of the groups list[0 .. nspin + nmain) of class CLS: the first nspin are the
// near-polar groups (spin form), the others run the plan's tuned shape in the scalar form
template <int CLS>
void leg_synth_cls(Plan &P, bool fp32, int nrhs, const int *list, int nspin, int nmain)
{
    if (fp32) leg_synth_s<float, CLS>(P, nrhs, list, nspin, nmain);
    else leg_synth_s<double, CLS>(P, nrhs, list, nspin, nmain);
}

// adjoint of the groups list[0 .. nspin + nmain): the spin groups into ring blocks rbs .., the others as
// split by sp (adj_split with this R, or RA, and W) into ring blocks rbm .. of nrb
template <typename S, int R, int W, int L, int CLS>
void adj_launch(Plan &P, int rhs, const int *list, int nspin, int nmain, const AdjSplit &sp, const uint8_t *live,
                int rbs, int rbm, int nrb)
{
    const int64_t fg_stride = (int64_t)P.nrings * (P.lmax + 1) * 2;
    const int nbs = (int)cdiv(nspin, spin_gpb(W));
    dim3 g((unsigned)(8 * (nbs + sp.q) * xcd_slots(P.lmax)));
    k_leg_adj<S, R, W, L, CLS><<<g, 64 * W, 0, P.stream>>>(
        (const cplx<S> *)P.d_FG + rhs * fg_stride, P.d_sa, P.d_coef64s, P.d_ent, P.d_entk, P.d_entl, P.ng64,
        P.d_pair_z, (S *)P.d_part, P.d_wgstart, P.next, P.lmax, P.npairs, P.nrings, list, nspin, nmain, live, rbs, rbm,
        nbs, sp.q, nrb, sp.nA);
}

// single-wave workgroups of at most RMAX groups, spread evenly (adj_split): the kernel of RA = sp.RA
// groups per workgroup, whose later workgroups take RA - 1
template <typename S, int RMAX, int L, int CLS>
void adj_launch_even(Plan &P, int rhs, const int *list, int nspin, int nmain, const AdjSplit &sp, const uint8_t *live,
                     int rbs, int rbm, int nrb)
{
    if constexpr (RMAX > 1) {
        if (sp.RA < RMAX)
            return adj_launch_even<S, RMAX - 1, L, CLS>(P, rhs, list, nspin, nmain, sp, live, rbs, rbm, nrb);
    }
    adj_launch<S, RMAX, 1, L, CLS>(P, rhs, list, nspin, nmain, sp, live, rbs, rbm, nrb);
}

// supported adjoint shapes (ring pairs per lane, waves per workgroup, l-chunk); the single-wave ones
// run through adj_launch_even
#define AKRA_ADJ_SHAPES_W1(X)                                                                          \
    X(1, 1, 8) X(2, 1, 8) X(3, 1, 8) X(4, 1, 8) X(5, 1, 8) X(6, 1, 8) X(7, 1, 8) X(8, 1, 8) X(1, 1, 4) X(2, 1, 4) \
        X(3, 1, 4) X(4, 1, 4) X(5, 1, 4) X(6, 1, 4) X(7, 1, 4) X(8, 1, 4)
#define AKRA_ADJ_SHAPES_WN(X) \
    X(1, 2, 8) X(1, 4, 8) X(2, 2, 8) X(2, 4, 8) X(4, 2, 8) X(4, 4, 8) X(8, 2, 8) X(2, 4, 4) X(4, 2, 4) X(4, 4, 4)
#define AKRA_ADJ_SHAPES(X) AKRA_ADJ_SHAPES_W1(X) AKRA_ADJ_SHAPES_WN(X)

// ring blocks of a class list's groups: those of nspin spin groups, and of nmain others (the class's tuned
// adj_R adj_W)
inline int adj_blocks_spin(const Plan &P, int cls, int nspin)
{
    int R, W, L;
    adj_shape_of(P, cls, R, W, L);
    return (int)cdiv(nspin, spin_gpb(W));
}
inline int adj_blocks_main(const Plan &P, int cls, int nmain)
{
    int R, W, L;
    adj_shape_of(P, cls, R, W, L);
    return adj_split(nmain, R, W).q;
}

template <typename S, int CLS>
void adj_dispatch(Plan &P, int rhs, const int *list, int nspin, int nmain, const uint8_t *live, int rbs, int rbm,
                  int nrb)
{
    int R, W, L;
    adj_shape_of(P, CLS, R, W, L);
    const AdjSplit sp = adj_split(nmain, R, W);
    if (W == 1) {
        if (nmain <= 0) return adj_launch<S, 1, 1, 8, CLS>(P, rhs, list, nspin, 0, sp, live, rbs, rbm, nrb);
        if (L == 4) return adj_launch_even<S, 8, 4, CLS>(P, rhs, list, nspin, nmain, sp, live, rbs, rbm, nrb);
        return adj_launch_even<S, 8, 8, CLS>(P, rhs, list, nspin, nmain, sp, live, rbs, rbm, nrb);
    }
#define AKRA_ADJ_CASE(r, w, l)        \
    if (R == r && W == w && L == l)   \
        return adj_launch<S, r, w, l, CLS>(P, rhs, list, nspin, nmain, sp, live, rbs, rbm, nrb);
    AKRA_ADJ_SHAPES_WN(AKRA_ADJ_CASE)
#undef AKRA_ADJ_CASE
}

// Legendre adjoint of right-hand side rhs over list[0 .. nspin + nmain) of class CLS: the near-polar
// groups into ring blocks rbs .., the others into ring blocks rbm .. of nrb
template <int CLS>
void leg_adj_cls(Plan &P, bool fp32, int rhs, const int *list, int nspin, int nmain, const uint8_t *live, int rbs,
                 int rbm, int nrb)
{
    if (fp32) adj_dispatch<float, CLS>(P, rhs, list, nspin, nmain, live, rbs, rbm, nrb);
    else adj_dispatch<double, CLS>(P, rhs, list, nspin, nmain, live, rbs, rbm, nrb);
}

extern template void leg_synth_cls<GCLS_BOTH>(Plan &, bool, int, const int *, int, int);
extern template void leg_synth_cls<GCLS_NORTH>(Plan &, bool, int, const int *, int, int);
extern template void leg_synth_cls<GCLS_SOUTH>(Plan &, bool, int, const int *, int, int);
extern template void leg_adj_cls<GCLS_BOTH>(Plan &, bool, int, const int *, int, int, const uint8_t *, int, int, int);
extern template void leg_adj_cls<GCLS_NORTH>(Plan &, bool, int, const int *, int, int, const uint8_t *, int, int, int);
extern template void leg_adj_cls<GCLS_SOUTH>(Plan &, bool, int, const int *, int, int, const uint8_t *, int, int, int);

}  // namespace akra
