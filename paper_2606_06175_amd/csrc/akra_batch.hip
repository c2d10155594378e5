// Batched Legendre kernels of FP32 plans with several right-hand sides (device code, gfx950): matrix
// products on the FP32 matrix cores with the recurrence values generated on the fly.
#include <type_traits>

#include "akra_leg.h"

namespace akra {
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

// exchange the upper half of a's lanes with the lower half of b's: a = [a_lo | b_lo], b = [a_hi | b_hi];
// and the odd rows (of 16 lanes) of a with the even rows of b
__device__ __forceinline__ void swap_halves(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
    a = __int_as_float(r[0]);
    b = __int_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
    a = __int_as_float(r[0]);
    b = __int_as_float(r[1]);
}

// ================================================================================================
// Scalar form (see akra_leg.h), groups of NB right-hand sides.  The four real sums of the scalar form per
// right-hand side are columns 4 rhs + c (c = Re q, Im q, Re u, Im u) of a matrix product
//   synthesis  [pairs x l] x [l x columns],      adjoint  [l x pairs] x [pairs x columns].
// The recurrence runs in FP64, one ring pair per lane (a multiply, an FMA and a conversion per degree;
// FP32 would need the coordinate as two floats, as many instructions, and its phase error sqrt(l) eps /
// theta dominated the transforms' error); the products and their sums are FP32.
//   NB = 8: v_mfma_f32_32x32x2_f32, 32 columns.   NB = 4: v_mfma_f32_16x16x4_f32, 16 columns, for groups of
//   at most four right-hand sides, which would leave half of the 32 columns empty.
// Bound by the matrix cores with the recurrence's vector work beside them (the two add up on this part,
// akra_mfma_rate): per pair and degree 4 columns a right-hand side, half of what the spin form needs,
// whose spin +2 and -2 functions each meet all four.
// Measured on a southern band of 0.35 of the sky, synthesis / adjoint per apply, spin form before -> now:
// Nside 512, lmax 1024, 4 right-hand sides 0.63 / 0.71 -> 0.22 / 0.35 ms (with NB = 8: 0.29 / 0.58 ms for the
// kernels alone, NB = 4: 0.17 / 0.35); Nside 1024, lmax 2048, 8 right-hand sides 3.6 / 3.9 -> 2.0 / 3.0 ms.
// Error of H x against FP64: 2.9e-6 -> 3.3e-7 and 3.5e-6 -> 4.2e-7.
// A operand of a product: row i in lane i + ROWS k; B operand: column j in lane j + COLS k.
// D: column lane % COLS, row drow(r, lane) of register r.
// ================================================================================================
template <int NB> struct Mf;
template <> struct Mf<8> {
    static constexpr int ROWS = 32, COLS = 32, K = 2, NR = 16;
    using acc = v16f;
    static __device__ __forceinline__ acc mul(float a, float b, acc d)
    {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, d, 0, 0, 0);
    }
    static __device__ __forceinline__ int drow(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
};
template <> struct Mf<4> {
    static constexpr int ROWS = 16, COLS = 16, K = 4, NR = 4;
    using acc = v4f;
    static __device__ __forceinline__ acc mul(float a, float b, acc d)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, d, 0, 0, 0);
    }
    static __device__ __forceinline__ int drow(int r, int lane) { return 4 * (lane >> 4) + r; }
};

// Records of one group: NB x 4 floats per entry (l, m), l <= lmax + 2, the stencil of k_prologue formed
// in FP64 and times c_l; zero past nrhs.  A workgroup takes 256 / NB entries; threads read along the
// entries of a right-hand side and the records go out through LDS in their own order.
template <int NB>
__global__ __launch_bounds__(256) void k_prologue_b(const double2 *__restrict__ xE, const double2 *__restrict__ xB,
                                                    int64_t rstride, const double *__restrict__ kern,
                                                    const uint32_t *__restrict__ lm, const double *__restrict__ sten,
                                                    const double *__restrict__ sc, int lmax, int64_t nalm,
                                                    int64_t next, int nrhs, int rhs0, float4 *__restrict__ brec)
{
    constexpr int NE = 256 / NB;
    __shared__ float4 sh[256];
    const int rr = threadIdx.x / NE, rhs = rhs0 + rr;
    const int64_t e0 = (int64_t)blockIdx.x * NE, e = e0 + threadIdx.x % NE;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (rhs < nrhs && e < next) {
        const int l = (int)(lm[e] & 0xffff), m = (int)(lm[e] >> 16);
        double q[4], K;
        double2 E, B;
        stencil_in(xE + rhs * rstride, xB + rhs * rstride, kern, sten, l, m, lmax, nalm, e - (int64_t)EXT_L * m, q, K,
                   E, B);
        const double s = sc[e];
        v = make_float4((float)(s * q[0]), (float)(s * q[1]), (float)(s * q[2]), (float)(s * q[3]));
    }
    sh[(threadIdx.x % NE) * NB + rr] = v;
    __syncthreads();
    if (e0 + threadIdx.x / NB < next) brec[e0 * NB + threadIdx.x] = sh[threadIdx.x];
}

// Synthesis: one wave per (m, 64-pair group), SW per workgroup.  Rounds of 2 K degrees: the values of the
// even and of the odd offsets from the entry degree are moved into the A layout by lane swaps (K = 2: one
// swap of wave halves per pair of degrees (l, l + 2); K = 4: a 4 x 4 transposition of rows and degrees
// l, l + 2, l + 4, l + 6), and each parity has 64 / ROWS accumulators, one per block of ROWS pairs.
template <int NB, int SW>
__global__ __launch_bounds__(64 * SW) void k_leg_synth_b(const float *__restrict__ brec, const double *__restrict__ sa,
                                                         float2 *__restrict__ FG, int64_t fg_stride,
                                                         const Ent64 *__restrict__ ent, const int *__restrict__ entk,
                                                         const int *__restrict__ entl, int ng64,
                                                         const double *__restrict__ pair_z, int lmax, int npairs,
                                                         int nrings, int nrhs, int rhs0,
                                                         const int *__restrict__ glist, int ngl, int nbm)
{
    using M = Mf<NB>;
    constexpr int DEG = 2 * M::K, PB = 64 / M::ROWS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int m, blk;
    xcd_map((int)blockIdx.x, nbm, m, blk);
    const int wi = blk * SW + wave;  // list entry of the wave
    if (m > lmax || wi >= ngl) return;
    const int g = uniform_ptr(glist)[wi];  // 64-pair group: pairs 64 g .. 64 g + 63
    const int lend = lmax + EXT_L;
    const int64_t base = ext_base(m, lmax);
    const int p = 64 * g + lane;
    // a group that never enters still writes its (zero) F
    const int ls = __builtin_amdgcn_readfirstlane(uniform_ptr(entl + (int64_t)m * ng64)[g]);
    double x = 0, c = 0, pv = 0;
    int k = 0;
    float f2 = 0.f;  // 1 / sin^2 of the lane's pair
    if (p < npairs) {
        x = pair_z[p];
        f2 = (float)(1.0 / ((1.0 - x) * (1.0 + x)));
        if (ls <= lend) load_entry_scalar(ent, entk, (int64_t)m * npairs + p, 0, c, pv, k);
    }
    typename M::acc D[2][PB];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < PB; ++b)
#pragma unroll
            for (int r = 0; r < M::NR; ++r) D[a][b][r] = 0.f;
    bool ramp = wave_any(k < 0);
    const_as<double> *cp = uniform_ptr(sa + base);
    const int kq = lane / M::COLS;
    const float *bl = brec + base * (NB * 4) + lane % M::COLS;  // the lane's column of the group's records
    // B rows l + 2 k (even offsets) and l + 1 + 2 k (odd) of a round; the buffer is padded
    struct Row {
        float e, o;
    };
    auto loadb = [&](int l) {
        const float *r = bl + (int64_t)(l + 2 * kq) * (NB * 4);
        return Row{r[0], r[NB * 4]};
    };
    // one round.  RAMP: some lane is still in the scaled range (its values count as zero until its
    // exponent reaches zero; the exponents are checked once per round); once no lane is, none returns to it
    auto round = [&](auto ramp_tag, const double *ca, const Row &r) {
        constexpr bool RAMP = decltype(ramp_tag)::value;
        float v[DEG];
#pragma unroll
        for (int t = 0; t < DEG; ++t) {
            v[t] = RAMP && k != 0 ? 0.f : (float)c;
            rstep_0(ca[t], x, c, pv);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            if constexpr (NB == 8) {
                swap_halves(v[a], v[2 + a]);
            } else {
                swap_halves(v[a], v[4 + a]);
                swap_halves(v[2 + a], v[6 + a]);
                swap_rows(v[a], v[2 + a]);
                swap_rows(v[4 + a], v[6 + a]);
            }
        }
#pragma unroll
        for (int b = 0; b < PB; ++b) {
            D[0][b] = M::mul(v[2 * b], r.e, D[0][b]);
            D[1][b] = M::mul(v[2 * b + 1], r.o, D[1][b]);
        }
        if constexpr (RAMP) {
            double z = 0;
            if (k < 0) rescale_slot<FORM_SCALAR>(c, pv, z, z, k);
            ramp = wave_any(k < 0);
        }
    };
    int l = ls <= lend ? ls : lend + 1;
    // four rounds per trip: each round's B rows are loaded into their registers four rounds ahead, and the
    // coefficients of two rounds after the first of the two before them (scalar loads return out of order:
    // one wait covers all in flight).  Loading them round by round, every round waited a memory latency (Nside 1024, lmax
    // 2048, 8 right-hand sides: 2.35 ms, so 1.73).
    Row rw[4];
    double cA[2 * DEG], cB[2 * DEG];
    auto loadc = [&](double (&cc)[2 * DEG], int l) {
#pragma unroll
        for (int t = 0; t < 2 * DEG; ++t) cc[t] = cp[l + t];
    };
#pragma unroll
    for (int t = 0; t < 4; ++t) rw[t] = loadb(l + t * DEG);
    loadc(cA, l);
    auto trip = [&](auto ramp_tag) {
        auto one = [&](int t, const double *cc) {
            round(ramp_tag, cc, rw[t]);
            rw[t] = loadb(l + (4 + t) * DEG);
            __builtin_amdgcn_sched_barrier(0);
        };
        one(0, cA);
        loadc(cB, l + 2 * DEG);
        __builtin_amdgcn_sched_barrier(0);
        one(1, cA + DEG);
        one(2, cB);
        loadc(cA, l + 4 * DEG);
        __builtin_amdgcn_sched_barrier(0);
        one(3, cB + DEG);
    };
    for (; l + 4 * DEG - 1 <= lend && ramp; l += 4 * DEG) trip(std::true_type{});
    for (; l + 4 * DEG - 1 <= lend; l += 4 * DEG) trip(std::false_type{});
    // the last rounds one by one, rows past the last degree as zero
    for (; l <= lend; l += DEG) {
        Row r = loadb(l);
        if (l + 2 * kq > lend) r.e = 0.f;
        if (l + 2 * kq + 1 > lend) r.o = 0.f;
        double ca[DEG];
#pragma unroll
        for (int t = 0; t < DEG; ++t) ca[t] = l + t <= lend ? cp[l + t] : 0.0;
        round(std::true_type{}, ca, r);
    }
    // F of the north (even + odd) and south (even - odd) ring of every (pair, rhs).  Lane c of a quad holds
    // S_c and gets S_{3-c}: F(m) = (S3 - S0, -(S1 + S2)), F(-m) = (-(S0 + S3), S1 - S2), times 1 / sin^2
    const int cc = lane & 3, rhs = rhs0 + lane % M::COLS / 4;
    float *Fb = (float *)(FG + (int64_t)rhs * fg_stride) + (cc ^ (cc >> 1));
#pragma unroll
    for (int b = 0; b < PB; ++b)
#pragma unroll
        for (int r = 0; r < M::NR; ++r) {
            const int i = b * M::ROWS + M::drow(r, lane), pi = 64 * g + i;
            const float f = __shfl(f2, i, 64);
            const float n = f * (D[0][b][r] + D[1][b][r]), s = f * (D[0][b][r] - D[1][b][r]);
            const float nx = dpp_mov<0x1B>(n), sx = dpp_mov<0x1B>(s);  // quad_perm [3, 2, 1, 0]
            if (rhs >= nrhs || pi >= npairs) continue;
            const int rs = nrings - 1 - pi;
            Fb[((int64_t)pi * (lmax + 1) + m) * 4] = (cc & 1) ? -(n + nx) : nx - n;
            if (rs != pi) Fb[((int64_t)rs * (lmax + 1) + m) * 4] = (cc & 1) ? -(s + sx) : sx - s;
        }
}

// Adjoint: for one m, a block of AW 64-pair groups (one per wave) and the right-hand sides of one group,
// the partial sums T_1, T_2 of the scalar form over the block's rings.  Per chunk of BCH = 64 degrees each
// wave writes the recurrence values of its pairs to LDS, the 32 even offsets and the 32 odd ones apart;
// the products of the even rows meet G of north + south, those of the odd rows north - south (both held in
// registers: they do not depend on l).  The waves of the block are summed in LDS and one slab per
// (right-hand side of the group, block) is written, [rhs - rhs0][nrb][next][4], rows from the chunk
// holding the block's first entry degree (recorded in wgstart) to lmax + 2.
// AW is a launch shape of the autotuner (2, 4 or 8): fewer waves in step with each other against more slabs for
// the epilogue.  Adjoint and epilogue of an iteration with four waves against two, footprint: Nside 256, 16 right-hand
// sides 36 us longer, Nside 512, four 23 us and 16 18 us longer, Nside 1024, eight 180 us and 16 390 us shorter (slabs
// dominate), which is what the autotuner finds.  Bound by the chunk's serial
// path (rows, operands, products, the sum of the waves): 0.38 of the FP32 matrix rate at Nside 512, 0.55 at 1024.
// Footprint, AW = 4: Nside 256, 16 right-hand sides 170 -> 102 us a group of eight with G loaded in
// batches and a' by vector loads (scalar loads without look-ahead before), Nside 512, four 373 -> 283 us.
constexpr int BCH = 64;                // degrees per chunk
template <int... I, typename F> __device__ __forceinline__ void static_for_(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    static_for_(std::make_integer_sequence<int, N>{}, f);
}
constexpr int BST = BCH / 2 + 1;       // LDS stride of one pair's rows of one parity (conflict-free writes)

template <int NB, int AW>
__global__ __launch_bounds__(64 * AW) __attribute__((amdgpu_waves_per_eu(2))) void k_leg_adj_b(
    const float2 *__restrict__ FG, int64_t fg_stride, const double *__restrict__ sa, const Ent64 *__restrict__ ent,
    const int *__restrict__ entk, const int *__restrict__ entl, int ng64, const double *__restrict__ pair_z,
    float *__restrict__ part, int *__restrict__ wgstart, int64_t slab, int lmax, int npairs, int nrings, int nrhs,
    int rhs0, const int *__restrict__ glist, int ngl, const uint8_t *__restrict__ live, int rb0, int nrbl, int nrb)
{
    using M = Mf<NB>;
    constexpr int NK = 64 / M::K, RBK = BCH / 2 / M::ROWS, NO = 2 * RBK * M::NR;
    __shared__ float lam[AW][2][64 * BST];  // per wave: rows of even and odd offsets of its 64 pairs
    __shared__ float red[8 * AW * 64];      // the cross-wave sum, eight output registers at a time
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int m, rbl;
    xcd_map((int)blockIdx.x, nrbl, m, rbl);
    if (m > lmax) return;
    const int rb = rb0 + rbl;
    const int lb = rbl * AW;  // first list entry of the block
    const int lend = lmax + EXT_L;
    const int64_t base = ext_base(m, lmax);
    const_as<int> *el = uniform_ptr(entl + (int64_t)m * ng64);
    const_as<int> *gl = uniform_ptr(glist);
    int ls = ENT_SKIP;
    for (int li = lb; li < lb + AW && li < ngl; ++li) ls = el[gl[li]] < ls ? el[gl[li]] : ls;
    if (threadIdx.x == 0) wgstart[(int64_t)m * nrb + rb] = ls;
    if (ls > lend) return;
    const int g = lb + wave < ngl ? gl[lb + wave] : -1;  // this wave's group
    const int e = g >= 0 ? el[g] : ENT_SKIP;             // and its entry degree
    const int p = g * 64 + lane;
    const bool valid = g >= 0 && p < npairs;

    // B operands: lane j + COLS k holds, for pairs K kk + k, column j of g_1, g_2 over sin^2.  Every lane
    // prepares 1 / 2 sin^2 and the weight flags of its own pair; the loads of G go out sixteen at a time,
    // none behind a condition (one pair after the other, with its position, flags and G in turn, they took
    // half of the kernel at Nside 256).
    const int kq = lane / M::COLS, j = lane % M::COLS, c4 = j & 3, rhs = rhs0 + j / 4;
    float Bp[NK], Bm[NK];
    double x = valid ? pair_z[p] : 0.0, c = 0, pv = 0;
    if (g >= 0 && e <= lend) {
        const double fz = 0.5 / ((1.0 - x) * (1.0 + x));
        const int rs = nrings - 1 - p;
        // a ring without weight has G = 0
        const uint64_t on_n = __ballot(valid && (!live || live[p]));
        const uint64_t on_s = __ballot(valid && rs != p && (!live || live[rs]));
        const float2 *F = FG + (int64_t)(rhs < nrhs ? rhs : nrhs - 1) * fg_stride + 2 * m;
        // columns: Re g_1 = (G.x + H.x) / 2, Im g_1 = (G.y - H.y) / 2, Re g_2 = (G.y + H.y) / 2,
        // Im g_2 = (H.x - G.x) / 2 with G = G(m), H = G(-m)
        auto comp = [&](float4 v, double f) {
            const double a = (c4 == 0 || c4 == 3) ? v.z : v.y;
            const double b = c4 == 0 ? v.x : c4 == 3 ? -v.x : c4 == 1 ? -v.w : v.w;
            return f * (a + b);
        };
#pragma unroll
        for (int k0 = 0; k0 < NK; k0 += 8) {
            float4 vn[8], vs[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int pk = g * 64 + M::K * (k0 + q) + kq, pc = pk < npairs ? pk : npairs - 1;
                vn[q] = *(const float4 *)(F + (int64_t)pc * (lmax + 1) * 2);
                vs[q] = *(const float4 *)(F + (int64_t)(nrings - 1 - pc) * (lmax + 1) * 2);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int i = M::K * (k0 + q) + kq;
                const double f = __shfl(fz, i, 64);
                const double n = rhs < nrhs && ((on_n >> i) & 1) ? comp(vn[q], f) : 0.0;
                const double s = rhs < nrhs && ((on_s >> i) & 1) ? comp(vs[q], f) : 0.0;
                Bp[k0 + q] = (float)(n + s);
                Bm[k0 + q] = (float)(n - s);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) Bp[kk] = Bm[kk] = 0.f;
    }

    int k = 0;
    bool ramp = false;
    // a' of the chunk at l: lane n of every row of 16 lanes holds degrees l + 16 i + n, a chunk ahead of
    // their use (DPP operands of the recurrence, in the signs of the single-vector synthesis)
    const double *cp = sa + base;
    auto loadc = [&](int l, double (&o)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int li = l + 16 * i + (lane & 15);
            o[i] = cp[li < lend ? li : lend];
        }
    };
    float *le = &lam[wave][0][lane * BST], *lo = &lam[wave][1][lane * BST];
    const int arow = lane / M::ROWS * BST + lane % M::ROWS;
    const float *ae = &lam[wave][0][arow], *ao = &lam[wave][1][arow];
    // the wave's recurrence covers the chunk starting at lx (zero before the wave's entry, for lanes
    // still in the scaled range and past the last degree)
    auto is_active = [&](int lx) { return lx <= lend && e <= lx + BCH - 1 && e <= lend; };
    // rows t8 .. t8 + 7 of the chunk at lx into the wave's LDS rows (entry degrees are m + 8 q and chunks
    // start at m + 64 j, so an entry falls on a block of 8)
    auto rows8 = [&](int lx, auto tc, const double (&cc)[4], auto &&after) {
        constexpr int t8 = decltype(tc)::value;
        const int l8 = lx + t8;
        if (l8 == e) {
            if (valid) load_entry_scalar(ent, entk, (int64_t)m * npairs + p, 0, c, pv, k);
            pv = -pv;
            ramp = wave_any(k < 0);
        }
        if (l8 < e || l8 > lend) {
            static_for<8>([&](auto t) {
                ((t & 1) ? lo : le)[(t8 + t) >> 1] = 0.f;
                after(t8 + t);
            });
            return;
        }
        auto step = [&](auto tc) {
            constexpr int t = decltype(tc)::value;
            const double xc = (t & 1) ? -x * c : x * c;
            // (the steps depend on each other, so the first one's wait covers the block; waiting by a volatile asm on
            // all of cc instead keeps the products from being scheduled across it: 5.05 against 4.70 ms at Nside 1024)
            if constexpr (t == 0) fma_row_settled<t8 % 16>(pv, cc[t8 / 16], xc);
            else fma_row<(t8 + t) % 16>(pv, cc[(t8 + t) / 16], xc);
            const double n = pv;
            pv = c;
            c = n;
        };
        if (!ramp && l8 + 7 <= lend) {
            // every lane out of the scaled range and every row in range: no selects, no checks
            static_for<8>([&](auto t) {
                ((t & 1) ? lo : le)[(t8 + t) >> 1] = (float)((t & 2) ? -c : c);
                step(t);
                after(t8 + t);
            });
            return;
        }
        static_for<8>([&](auto t) {
            ((t & 1) ? lo : le)[(t8 + t) >> 1] = k == 0 && l8 + t <= lend ? (float)((t & 2) ? -c : c) : 0.f;
            step(t);
            after(t8 + t);
        });
        // every eight steps (the growth over eight steps stays far from overflow)
        double z = 0;
        if (k < 0) rescale_slot<FORM_SCALAR>(c, pv, z, z, k);
        ramp = wave_any(k < 0);
    };
    auto rows = [&](int lx, const double (&cc)[4], auto &&after) {
        static_for<BCH / 8>([&](auto i) { rows8(lx, std::integral_constant<int, 8 * decltype(i)::value>{}, cc, after); });
    };
    // Software pipeline over chunks: the A operands of chunk lc are read from LDS into registers, then
    // the recurrence writes the rows of the next chunk into the same LDS rows while the matrix cores
    // contract chunk lc, one product per row.  A wave reads and writes only its own rows, and its LDS
    // accesses run in program order, so the reads return the rows of chunk lc.
    const int lstart = m + ((ls - m) / BCH) * BCH;
    double cc[4], cn[4];
    loadc(lstart, cc);
    loadc(lstart + BCH, cn);
    if (is_active(lstart)) rows(lstart, cc, [](int) {});
    for (int lc = lstart; lc <= lend; lc += BCH) {
#pragma unroll
        for (int i = 0; i < 4; ++i) cc[i] = cn[i];
        loadc(lc + 2 * BCH, cn);
        const bool act = is_active(lc), actn = is_active(lc + BCH);
        wg_lds_sync<1>();
        float a[2][RBK][NK];
        if (act) {
#pragma unroll
            for (int kk = 0; kk < NK; ++kk)
#pragma unroll
                for (int b = 0; b < RBK; ++b) {
                    a[0][b][kk] = ae[M::K * kk * BST + b * M::ROWS];
                    a[1][b][kk] = ao[M::K * kk * BST + b * M::ROWS];
                }
        }
        wg_lds_sync<1>();
        typename M::acc D[2][RBK];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int b = 0; b < RBK; ++b)
#pragma unroll
                for (int r = 0; r < M::NR; ++r) D[q][b][r] = 0.f;
        // product i of the chunk's 2 RBK NK = 64
        auto mm = [&](int i) {
            const int q = i & 1, b = (i >> 1) % RBK, kk = (i >> 1) / RBK;
            D[q][b] = M::mul(a[q][b][kk], q ? Bm[kk] : Bp[kk], D[q][b]);
        };
        static_assert(2 * RBK * NK == BCH, "one product per row");
        if (act && actn) {
            rows(lc + BCH, cc, [&](int i) { mm(i); });
        } else if (act) {
#pragma unroll
            for (int i = 0; i < BCH; ++i) mm(i);
        } else if (actn) {
            rows(lc + BCH, cc, [](int) {});
        }
        // sum over the block's waves in LDS, eight registers at a time
        float o[NO];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int b = 0; b < RBK; ++b)
#pragma unroll
                for (int r = 0; r < M::NR; ++r) o[(q * RBK + b) * M::NR + r] = D[q][b][r];
#pragma unroll
        for (int h = 0; h < NO; h += 8) {
            __syncthreads();
#pragma unroll
            for (int r8 = 0; r8 < 8; ++r8) red[(wave * 8 + r8) * 64 + lane] = o[h + r8];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 8 / AW; ++u) {
                const int r = h + wave * (8 / AW) + u;  // this thread's register index, lane as it was
                float sum = 0.f;
#pragma unroll
                for (int w = 0; w < AW; ++w) sum += red[(w * 8 + r - h) * 64 + lane];
                const int q = r / (RBK * M::NR), b = r / M::NR % RBK;
                const int l = lc + 2 * (b * M::ROWS + M::drow(r % M::NR, lane)) + q;
                if (l <= lend && rhs < nrhs) part[(((int64_t)(j / 4) * nrb + rb) * slab + base + l) * 4 + c4] = sum;
            }
        }
    }
}

// ================================================================================================
// Spin form of the groups that begin within AKRA_POLE_THETA_B radians of a pole: NBR = 8 right-hand
// sides per group, the spin-weighted functions in the FP32 difference form.
// Synthesis: for one m, a group of 64 ring pairs
// (one per lane) and NBR = 8 right-hand sides, the sums over l of lambda(l, pair) a(l, rhs, c) are a
// matrix product [pairs x l] x [l x (rhs, c)] with the lambda generated on the fly, accumulated on
// the matrix cores (v_mfma_f32_32x32x2_f32: D[32 x 32] += A[32 x 2] B[2 x 32]), per half of the pairs.
//   A[i][k]  lambda of pair i (of the half) at degree l + 2k (even offsets from the step l of four) or
//            l + 1 + 2k (odd), held by lane i + 32k.  Every lane runs the recurrence of its own pair;
//            one v_permlane32_swap per pair of degrees (l, l+2) moves the values into that layout:
//            [low lanes at l | low lanes at l+2] for the first half, [high at l | high at l+2] for
//            the second.
//   B[k][j]  record value j = 4 rhs + c (c = Re/Im of aE, Re/Im of aB) at the same degree
//   D        per half four accumulators: spin +2 / -2 times even / odd offsets from the start degree
// Lane l, register r of D holds pair i = 8 (r/4) + 4 (l/32) + r%4 of the half and column j = l%32.
// ================================================================================================
// spin form, per (l, m): the NBR x 4 kernel-scaled alm values of one group (Im(a_l0) zeroed), zero past nrhs
__global__ void k_prologue_spin_b(const double *__restrict__ xE, const double *__restrict__ xB, int64_t rstride,
                             const double *__restrict__ kern, const int *__restrict__ lof, int lmax, int64_t nalm,
                             int nrhs, int q, float *__restrict__ brec)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // (alm, rhs-in-group)
    if (t >= nalm * NBR) return;
    const int64_t i = t / NBR;
    const int rr = (int)(t - i * NBR), rhs = q * NBR + rr;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (rhs < nrhs) {
        const int64_t o = (int64_t)rhs * rstride + i;  // rstride: complex elements between right-hand sides
        const double K = kern ? kern[lof[i]] : 1.0;
        const bool m0 = i <= lmax;
        v.x = (float)(K * xE[2 * o]);
        v.y = m0 ? 0.f : (float)(K * xE[2 * o + 1]);
        v.z = (float)(K * xB[2 * o]);
        v.w = m0 ? 0.f : (float)(K * xB[2 * o + 1]);
    }
    reinterpret_cast<float4 *>(brec)[t] = v;
}

// quad sum over the four lanes 4 rhs + (0..3) that hold c = 0..3 of one right-hand side
__device__ __forceinline__ float quad_sum(float v)
{
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    return v;
}

template <int SW>
__global__ __launch_bounds__(64 * SW) __attribute__((amdgpu_waves_per_eu(2))) void k_spin_synth_b(const float *__restrict__ brec,
                                                     const Coef32D *__restrict__ coef,
                                                     float2 *__restrict__ FG, int64_t fg_stride,
                                                     const Ent64 *__restrict__ ent, const int *__restrict__ entk,
                                                     const int *__restrict__ entl, int ng64,
                                                     const double *__restrict__ pair_z, int lmax, int npairs,
                                                     int nrings, int nrhs, int q, const int *__restrict__ glist,
                                                     int ngl, int nbm)
{
    const int lane = threadIdx.x & 63, h = lane >> 5, i = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int m, blk;
    xcd_map((int)blockIdx.x, nbm, m, blk);
    const int wi = blk * SW + wave;  // list entry of the wave
    if (m > lmax || wi >= ngl) return;
    const int w = uniform_ptr(glist)[wi];  // 64-pair group: pairs 64 w .. 64 w + 63
    const int l0 = m > 2 ? m : 2;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    const int p = 64 * w + lane;
    // a group that never enters still writes its (zero) F
    const int ls = __builtin_amdgcn_readfirstlane(uniform_ptr(entl + (int64_t)m * ng64)[w]);

    YF x;
    float c2 = 0.f, p2 = 0.f, cm = 0.f, pm = 0.f;
    int k = 0;
    setpos(x, 0.0);
    if (p < npairs && ls <= lmax) {
        setpos(x, pair_z[p]);
        load_entry_b(ent, entk, (int64_t)m * npairs + p, c2, p2, cm, pm, k);
    }
    v16f D2e[2], D2o[2], Dme[2], Dmo[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int r = 0; r < 16; ++r) D2e[s2][r] = D2o[s2][r] = Dme[s2][r] = Dmo[s2][r] = 0.f;
    bool ramp = wave_any(k < 0);
    using C = Coef32D;
    const_as<C> *cp = uniform_ptr(coef + base);
    const float *bl = brec + base * (NBR * 4) + i;  // column i of the group's records
    // four degrees from l: records and recurrence values, then the eight products.  RAMP: some lane is
    // still in the scaled range (its values count as zero until its exponent reaches zero, and the
    // exponents are checked once per four steps); once no lane is, none returns to it, and the loop
    // without the selects and the checks takes over.
    auto four = [&](int l, auto ramp_tag) {
        constexpr bool RAMP = decltype(ramp_tag)::value;
        // B rows l + 2h (even offsets) and l + 1 + 2h (odd), zero past lmax
        const int re = l + 2 * h, ro = re + 1;
        const float be = re <= lmax ? bl[(int64_t)re * (NBR * 4)] : 0.f;
        const float bo = ro <= lmax ? bl[(int64_t)ro * (NBR * 4)] : 0.f;
        float v2[4], vm[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const bool live = !RAMP || k == 0;
            v2[t] = live ? c2 : 0.f;
            vm[t] = live ? cm : 0.f;
            rstep(ld_coef(cp + l + t), x, c2, p2, cm, pm);
        }
        // degrees (l, l+2) and (l+1, l+3) of both halves of the pairs
        swap_halves(v2[0], v2[2]);
        swap_halves(v2[1], v2[3]);
        swap_halves(vm[0], vm[2]);
        swap_halves(vm[1], vm[3]);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            D2e[s2] = __builtin_amdgcn_mfma_f32_32x32x2f32(v2[2 * s2], be, D2e[s2], 0, 0, 0);
            D2o[s2] = __builtin_amdgcn_mfma_f32_32x32x2f32(v2[2 * s2 + 1], bo, D2o[s2], 0, 0, 0);
            Dme[s2] = __builtin_amdgcn_mfma_f32_32x32x2f32(vm[2 * s2], be, Dme[s2], 0, 0, 0);
            Dmo[s2] = __builtin_amdgcn_mfma_f32_32x32x2f32(vm[2 * s2 + 1], bo, Dmo[s2], 0, 0, 0);
        }
        if constexpr (RAMP) {
            // once per four steps (the growth over four steps stays far from overflow)
            if (k < 0 && fmaxf(fabsf(c2), fabsf(cm)) > scale_hi<float>()) {
                const float d = scale_down<float>();
                c2 *= d;
                p2 *= d;
                cm *= d;
                pm *= d;
                k += 1;
            }
            ramp = wave_any(k < 0);
        }
    };
    int l = ls;
    for (; l <= lmax && ramp; l += 4) four(l, std::true_type{});
    for (; l <= lmax; l += 4) four(l, std::false_type{});
    // F of the north and south ring of every (pair, rhs): quad sums over c, written by lane c = 0
    const bool odd0 = ((l0 + m) & 1) != 0;  // entries are l0 + 8 q: D2e holds degrees of parity l0 + m
    const int c = i & 3, rl = i >> 2, rhs = q * NBR + rl;
    const float s0r = c == 0 ? -1.f : (c == 3 ? 1.f : 0.f), s0i = (c == 1 || c == 2) ? -1.f : 0.f;
    const float s1r = (c == 0 || c == 3) ? -1.f : 0.f, s1i = c == 2 ? -1.f : (c == 1 ? 1.f : 0.f);
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int pi = 64 * w + 32 * s2 + 8 * (r >> 2) + 4 * h + (r & 3);
            const float E2 = odd0 ? D2o[s2][r] : D2e[s2][r], O2 = odd0 ? D2e[s2][r] : D2o[s2][r];
            const float Em = odd0 ? Dmo[s2][r] : Dme[s2][r], Om = odd0 ? Dme[s2][r] : Dmo[s2][r];
            // north: S2 = E2 + O2, Sm = Em + Om;  south: S2 = Em - Om, Sm = E2 - O2
            const float S2n = E2 + O2, Smn = Em + Om, S2s = Em - Om, Sms = E2 - O2;
            // f0 = -(S2[0] - S2[3], S2[1] + S2[2]),  f1 = -(Sm[0] + Sm[3], Sm[2] - Sm[1])
            const float fn0r = quad_sum(s0r * S2n), fn0i = quad_sum(s0i * S2n);
            const float fn1r = quad_sum(s1r * Smn), fn1i = quad_sum(s1i * Smn);
            const float fs0r = quad_sum(s0r * S2s), fs0i = quad_sum(s0i * S2s);
            const float fs1r = quad_sum(s1r * Sms), fs1i = quad_sum(s1i * Sms);
            if (c == 0 && rhs < nrhs && pi < npairs) {
                float2 *Fb = FG + (int64_t)rhs * fg_stride;
                const int rn = pi, rs = nrings - 1 - pi;
                float2 *f = Fb + ((int64_t)rn * (lmax + 1) + m) * 2;
                f[0] = make_float2(fn0r, fn0i);
                f[1] = make_float2(fn1r, fn1i);
                if (rs != rn) {
                    float2 *g = Fb + ((int64_t)rs * (lmax + 1) + m) * 2;
                    g[0] = make_float2(fs0r, fs0i);
                    g[1] = make_float2(fs1r, fs1i);
                }
            }
        }
    }
}

// ================================================================================================
// Batched FP32 Legendre adjoint on the matrix cores.  For one m, a block of AW 64-pair groups (one per
// wave) and the NBR right-hand sides of group q, the partial sums over the block's ring pairs
//   out_rhs[l][c],  c = 0..3 as in k_leg_adj (2h_lm and -2h_lm, Re and Im).
// Per chunk of ABL = 32 degrees each wave writes the recurrence values of its pairs to LDS (one row
// per degree), then v_mfma_f32_32x32x2_f32 contracts over the pairs, two per instruction:
//   D+ = Lambda+ [GN.x, GN.y, HS.x, HS.y],   D- = Lambda- [HN.x, HN.y, GS.x, GS.y]
// (columns 4 rhs + c, G of the north ring GN, HN = conj of its second component, S the south ring),
// and the south terms take the sign s = (-1)^(l+m) of their row:
//   out_0,1 = D+[c] + s D-[c+2],   out_2,3 = D-[c-2] + s D+[c].
// G is loaded once per wave into registers (it does not depend on l).  The waves of the block are
// summed in LDS and one slab per (right-hand side of the group, block) is written,
// [rhs - NBR q][nrb][next][4] (nalm rows used), rows from the chunk holding the block's first entry degree (recorded in
// wgstart) to lmax.
// ================================================================================================
// AW waves (64-pair groups) per workgroup is a launch shape of the autotuner (2, 4 or 8)
constexpr int ABL = 32;  // degrees per chunk: the rows of the MFMA
constexpr int ABS = 33;  // LDS stride of one pair's 32 rows (bank-conflict-free writes)

template <int AW>
__global__ __launch_bounds__(64 * AW) __attribute__((amdgpu_waves_per_eu(2))) void k_spin_adj_b(const float2 *__restrict__ FG, int64_t fg_stride,
                                                        const Coef32D *__restrict__ coef,
                                                        const Ent64 *__restrict__ ent, const int *__restrict__ entk,
                                                        const int *__restrict__ entl, int ng64,
                                                        const double *__restrict__ pair_z, float *__restrict__ part,
                                                        int *__restrict__ wgstart, int lmax, int npairs,
                                                        int nrings, int nrhs, int q, const int *__restrict__ glist,
                                                        int ngl, const uint8_t *__restrict__ live, int rb0,
                                                        int nrbl, int nrb, int64_t slab)
{
    __shared__ float lam[AW][2][64 * ABS];  // per wave: lambda+ and lambda- of its 64 pairs x 32 rows
    __shared__ float red[8 * AW * 64];      // the cross-wave sum, eight output registers at a time
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int m, rbl;
    xcd_map((int)blockIdx.x, nrbl, m, rbl);
    if (m > lmax) return;
    const int rb = rb0 + rbl;
    const int lb = rbl * AW;  // first list entry of the block
    const int l0 = m > 2 ? m : 2;
    const int64_t base = (int64_t)m * (2 * lmax + 1 - m) / 2;
    const_as<int> *el = uniform_ptr(entl + (int64_t)m * ng64);
    const_as<int> *gl = uniform_ptr(glist);
    int ls = ENT_SKIP;
    for (int li = lb; li < lb + AW && li < ngl; ++li) ls = el[gl[li]] < ls ? el[gl[li]] : ls;
    if (threadIdx.x == 0) wgstart[(int64_t)m * nrb + rb] = ls;
    if (ls > lmax) return;
    const int g = lb + wave < ngl ? gl[lb + wave] : -1;  // this wave's group
    const int e = g >= 0 ? el[g] : ENT_SKIP;             // and its entry degree
    const int p = g * 64 + lane;
    const bool valid = g >= 0 && p < npairs;

    // B operands: lane l holds, for pair-pair kk, pair 64 g + 2 kk + l / 32 and column j = l % 32
    const int j = lane & 31, c = j & 3, rhs = q * NBR + (j >> 2);
    float Bp[32], Bm[32];
#pragma unroll
    for (int kk = 0; kk < 32; ++kk) {
        Bp[kk] = Bm[kk] = 0.f;
        const int pk = g * 64 + 2 * kk + (lane >> 5);
        if (e > lmax || g < 0 || pk >= npairs || rhs >= nrhs) continue;
        const float2 *Fb = FG + rhs * fg_stride;
        if (c < 2) {
            if (live && !live[pk]) continue;  // a ring without weight has G = 0
            const float2 *fn = Fb + ((int64_t)pk * (lmax + 1) + m) * 2;
            const float2 gn = fn[0], hn = fn[1];  // HN = conj(hn)
            Bp[kk] = c ? gn.y : gn.x;
            Bm[kk] = c ? -hn.y : hn.x;
        } else {
            const int rs = nrings - 1 - pk;
            if (rs != pk && (!live || live[rs])) {
                const float2 *fs = Fb + ((int64_t)rs * (lmax + 1) + m) * 2;
                const float2 gs = fs[0], hs = fs[1];  // HS = conj(hs)
                Bp[kk] = (c & 1) ? -hs.y : hs.x;
                Bm[kk] = (c & 1) ? gs.y : gs.x;
            }
        }
    }

    YF x;
    setpos(x, valid ? pair_z[p] : 0.0);
    float c2 = 0.f, p2 = 0.f, cm = 0.f, pm = 0.f;
    int k = 0;
    bool ramp = false;
    using C = Coef32D;
    const_as<C> *cp = uniform_ptr(coef + base);
    float *lp = &lam[wave][0][lane * ABS], *lmn = &lam[wave][1][lane * ABS];
    const float *ap = &lam[wave][0][(lane >> 5) * ABS + (lane & 31)], *am = &lam[wave][1][(lane >> 5) * ABS + (lane & 31)];
    // the wave's recurrence covers the chunk starting at lx (zero before the wave's entry, for lanes
    // still in the scaled range and past lmax)
    auto is_active = [&](int lx) { return lx <= lmax && e <= lx + ABL - 1 && e <= lmax; };
    // rows t8 .. t8 + 7 of the chunk at lx into the wave's LDS rows (entry degrees are l0 + 8 q and
    // chunks start at l0 + 32 j, so an entry falls on a block of 8)
    auto rows8 = [&](int lx, int t8, auto &&after) {
        const int lb = lx + t8;
        if (lb == e) {
            if (valid) load_entry_b(ent, entk, (int64_t)m * npairs + p, c2, p2, cm, pm, k);
            ramp = wave_any(k < 0);
        }
        if (lb < e || lb > lmax) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                lp[t8 + t] = lmn[t8 + t] = 0.f;
                after(t);
            }
            return;
        }
        C cc[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) cc[t] = ld_coef(cp + lb + t);  // padded past lmax
        if (!ramp && lb + 7 <= lmax) {
            // every lane out of the scaled range and every row in range: no selects, no checks
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                lp[t8 + t] = c2;
                lmn[t8 + t] = cm;
                rstep(cc[t], x, c2, p2, cm, pm);
                after(t);
            }
            return;
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const bool live = k == 0 && lb + t <= lmax;
            lp[t8 + t] = live ? c2 : 0.f;
            lmn[t8 + t] = live ? cm : 0.f;
            rstep(cc[t], x, c2, p2, cm, pm);
            after(t);
            if (ramp && (t & 3) == 3) {
                // every four steps (the growth over four steps stays far from overflow)
                if (k < 0 && fmaxf(fabsf(c2), fabsf(cm)) > scale_hi<float>()) {
                    const float d = scale_down<float>();
                    c2 *= d;
                    p2 *= d;
                    cm *= d;
                    pm *= d;
                    k += 1;
                }
                ramp = wave_any(k < 0);
            }
        }
    };
    // Software pipeline over chunks: the A operands of chunk lc are read from LDS into registers, then
    // the recurrence writes the rows of the next chunk into the same LDS rows while the matrix cores
    // contract chunk lc (eight rows, then the sixteen products of eight pair-pairs).  A wave reads and
    // writes only its own rows, and its LDS accesses run in program order, so the reads return the
    // rows of chunk lc.
    const int lstart = l0 + ((ls - l0) / ABL) * ABL;
    if (is_active(lstart)) {
#pragma unroll
        for (int t8 = 0; t8 < ABL; t8 += 8) rows8(lstart, t8, [](int) {});
    }
    for (int lc = lstart; lc <= lmax; lc += ABL) {
        const bool act = is_active(lc), actn = is_active(lc + ABL);
        wg_lds_sync<1>();
        float a[32], b[32];
        if (act) {
#pragma unroll
            for (int kk = 0; kk < 32; ++kk) {
                a[kk] = ap[2 * kk * ABS];
                b[kk] = am[2 * kk * ABS];
            }
        }
        wg_lds_sync<1>();
        v16f Dp, Dm;
#pragma unroll
        for (int r = 0; r < 16; ++r) Dp[r] = Dm[r] = 0.f;
        // the products of pair-pair kk follow row kk % 8 of block kk / 8 of the next chunk
        auto mm = [&](int kk) {
            Dp = __builtin_amdgcn_mfma_f32_32x32x2f32(a[kk], Bp[kk], Dp, 0, 0, 0);
            Dm = __builtin_amdgcn_mfma_f32_32x32x2f32(b[kk], Bm[kk], Dm, 0, 0, 0);
        };
        if (act && actn) {
#pragma unroll
            for (int t8 = 0; t8 < ABL; t8 += 8) rows8(lc + ABL, t8, [&](int t) { mm(t8 + t); });
        } else if (act) {
#pragma unroll
            for (int kk = 0; kk < 32; ++kk) mm(kk);
        } else if (actn) {
#pragma unroll
            for (int t8 = 0; t8 < ABL; t8 += 8) rows8(lc + ABL, t8, [](int) {});
        }
        // D row of register r in lane l: 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
        float o[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            const float s = ((lc + i + m) & 1) ? -1.f : 1.f;
            const float t2 = dpp_mov<0x4E>(Dm[r]);  // D- of column j ^ 2
            o[r] = c < 2 ? fmaf(s, t2, Dp[r]) : fmaf(s, Dp[r], t2);
        }
        // sum over the block's waves in LDS, eight registers at a time
#pragma unroll
        for (int h = 0; h < 16; h += 8) {
            __syncthreads();
#pragma unroll
            for (int r8 = 0; r8 < 8; ++r8) red[(wave * 8 + r8) * 64 + lane] = o[h + r8];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 8 / AW; ++u) {
                const int r = h + wave * (8 / AW) + u;  // this thread's register index, lane as it was
                float sum = 0.f;
#pragma unroll
                for (int w = 0; w < AW; ++w) sum += red[(w * 8 + r - h) * 64 + lane];
                const int i = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), l = lc + i;
                if (l <= lmax && rhs < nrhs)
                    part[(((int64_t)(j >> 2) * nrb + rb) * slab + base + l) * 4 + c] = sum;
            }
        }
    }
}

// near-polar and other groups (n1, n2 of them) touch disjoint rings and slabs: the near-polar launch, few
// waves with long recurrences, runs beside the other
template <class A, class B> static void beside(Plan &P, int n1, int n2, A &&pol, B &&rest)
{
    if (n1 > 0 && n2 > 0) return fork_join(P, pol, rest);
    if (n1 > 0) pol();
    if (n2 > 0) rest();
}

// groups of at most NBR right-hand sides: the matrix-core shape of group q
static int group_nb(const Plan &P, int q) { return P.nrhs - NBR * q <= 4 ? 4 : 8; }

template <int NB, int SW>
static void synth_b_launch(Plan &P, int q, int64_t fg_stride, const int *list, int n)
{
    const int nbm = (int)cdiv(n, SW);
    k_leg_synth_b<NB, SW><<<(unsigned)(8 * nbm * xcd_slots(P.lmax)), 64 * SW, 0, P.stream>>>(
        P.d_brec, P.d_sa, (float2 *)P.d_FG, fg_stride, P.d_ent, P.d_entk, P.d_entl, P.ng64, P.d_pair_z, P.lmax,
        P.npairs, P.nrings, P.nrhs, NBR * q, list, n, nbm);
}

template <int SW> static void spin_synth_b_launch(Plan &P, int q, int64_t fg_stride, const int *list, int n)
{
    const int nbm = (int)cdiv(n, SW);
    k_spin_synth_b<SW><<<(unsigned)(8 * nbm * xcd_slots(P.lmax)), 64 * SW, 0, P.stream>>>(
        P.d_brec_spin, P.d_coef32d, (float2 *)P.d_FG, fg_stride, P.d_ent, P.d_entk, P.d_entl, P.ng64, P.d_pair_z,
        P.lmax, P.npairs, P.nrings, P.nrhs, q, list, n, nbm);
}

template <int AW>
static void adj_b_launch(Plan &P, int q, int64_t fg_stride, const int *list, int npol, int nmain, const uint8_t *live,
                         int nrb)
{
    const int64_t slots = xcd_slots(P.lmax);
    const int nbp = (int)cdiv(npol, AW), nbn = (int)cdiv(nmain, AW);
    auto pol = [&]() {
        k_spin_adj_b<AW><<<(unsigned)(8 * nbp * slots), 64 * AW, 0, P.stream>>>(
            (const float2 *)P.d_FG, fg_stride, P.d_coef32d, P.d_ent, P.d_entk, P.d_entl, P.ng64, P.d_pair_z,
            (float *)P.d_part, P.d_wgstart_b, P.lmax, P.npairs, P.nrings, P.nrhs, q, list, npol, live, 0, nbp,
            nrb, P.next);
    };
    auto main = [&](auto kern) {
        kern<<<(unsigned)(8 * nbn * slots), 64 * AW, 0, P.stream>>>(
            (const float2 *)P.d_FG, fg_stride, P.d_sa, P.d_ent, P.d_entk, P.d_entl, P.ng64, P.d_pair_z,
            (float *)P.d_part, P.d_wgstart_b, P.next, P.lmax, P.npairs, P.nrings, P.nrhs, NBR * q, list + npol, nmain,
            live, nbp, nbn, nrb);
    };
    auto rest = [&]() {
        if (group_nb(P, q) == 4) main(k_leg_adj_b<4, AW>);
        else main(k_leg_adj_b<8, AW>);
    };
    beside(P, nbp, nbn, pol, rest);
}

// batched synthesis of FP32 plans: records and matrix-core sums per group of NBR right-hand sides, over
// every 64-pair group (live false) or those with a ring that carries weight (live true)
void launch_synth_batched(Plan &P, const double *xE, const double *xB, int64_t rstride, const double *kern, bool live)
{
    const int64_t fg_stride = (int64_t)P.nrings * (P.lmax + 1) * 2;
    const GroupSet &G = live && P.skip_rings ? P.gs_live : P.gs_all;
    const int *pol = G.list_any, *rest = G.list_any + G.npol_any;
    for (int q = 0; q * NBR < P.nrhs; ++q) {
        const bool four = group_nb(P, q) == 4;
        auto pro = [&](auto kern_b, int nb) {
            kern_b<<<(unsigned)cdiv(P.next, 256 / nb), 256, 0, P.stream>>>(
                (const double2 *)xE, (const double2 *)xB, rstride, kern, P.d_lm, P.d_sten, P.d_sc, P.lmax, P.nalm,
                P.next, P.nrhs, NBR * q, (float4 *)P.d_brec);
        };
        if (four) pro(k_prologue_b<4>, 4);
        else pro(k_prologue_b<8>, 8);
        if (G.npol_any > 0)
            k_prologue_spin_b<<<(unsigned)cdiv(P.nalm * NBR, 256), 256, 0, P.stream>>>(
                xE, xB, rstride, kern, P.d_lof, P.lmax, P.nalm, P.nrhs, q, P.d_brec_spin);
        auto run = [&](auto sw) {
            constexpr int SW = decltype(sw)::value;
            beside(P, G.npol_any, G.nmain_any, [&]() { spin_synth_b_launch<SW>(P, q, fg_stride, pol, G.npol_any); },
                   [&]() {
                       if (four) synth_b_launch<4, SW>(P, q, fg_stride, rest, G.nmain_any);
                       else synth_b_launch<8, SW>(P, q, fg_stride, rest, G.nmain_any);
                   });
        };
        switch (P.bat_SW) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 8: run(std::integral_constant<int, 8>{}); break;
        default: run(std::integral_constant<int, 4>{});
        }
    }
}

// batched adjoint of the right-hand-side group q into the [rhs - NBR q][nrb_b_cur][next][4] slabs of
// d_part (the first nrbs_b_cur in the spin form), over every 64-pair group (live false) or those with a
// ring that carries weight, reading only such rings (live true)
void launch_adj_batched(Plan &P, int q, bool live)
{
    live = live && P.skip_rings;
    const int64_t fg_stride = (int64_t)P.nrings * (P.lmax + 1) * 2;
    const GroupSet &G = live ? P.gs_live : P.gs_all;
    const uint8_t *lv = live ? P.d_ring_live : nullptr;
    const int nbp = (int)cdiv(G.npol_any, P.bat_AW), nrb = nbp + (int)cdiv(G.nmain_any, P.bat_AW);
    switch (P.bat_AW) {
    case 2: adj_b_launch<2>(P, q, fg_stride, G.list_any, G.npol_any, G.nmain_any, lv, nrb); break;
    case 8: adj_b_launch<8>(P, q, fg_stride, G.list_any, G.npol_any, G.nmain_any, lv, nrb); break;
    default: adj_b_launch<4>(P, q, fg_stride, G.list_any, G.npol_any, G.nmain_any, lv, nrb);
    }
    P.nrb_b_cur = nrb;
    P.nrbs_b_cur = nbp;
}

}  // namespace akra
