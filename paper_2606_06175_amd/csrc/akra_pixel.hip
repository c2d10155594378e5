// Catalogue pixelisation (Sec. III.B pixelization): galaxies binned onto the HEALPix RING grid, and
// per pixel the weighted shear (eq. gamma_obs), the effective count N_eff (eq. Neff_pixel), the
// inverse noise N^-1 = N_eff / sigma_e^2 (eq. noise_var) and the threshold mask (eq. mask).
//
// The sums of a pixel run over its galaxies in catalogue order with contraction off: up to BUCKET_NPIX
// pixels a stable partition brings the galaxies of each pixel range together and a workgroup per range adds
// them in order in LDS; beyond, a stable radix sort of (pixel, galaxy) pairs groups them and one thread
// per pixel accumulates sequentially.  Every output is therefore a fixed, IEEE-rounded function of the catalogue -- no atomics,
// no dependence on scheduling -- and the threshold decision N_eff >= N_th is reproducible.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/iterator/counting_iterator.hpp>

#include "akra_internal.h"

namespace akra {

// RING index of the direction (z = cos theta, phi in [0, 2 pi)) from the inverse of the HEALPix
// pixel boundaries (Gorski et al. 2005): in the equatorial belt |z| <= 2/3 the pixel edges are the
// lines Nside (1/2 + t) -+ (3/4) Nside z of t = phi / (pi/2), whose integer parts jp, jm give the
// ring ir = Nside + 1 + jp - jm (counted from z = 2/3) and the position in it; in the caps the edges
// are f h and (1 - f) h with f = frac(t), h = Nside sqrt(3 (1 - |z|)), giving the ring from the pole
// ir = jp + jm + 1 and the position floor(t ir) mod 4 ir.  Each product and sum is rounded on its own.
__device__ int64_t ang2pix_ring(int nside, double z, double phi)
{
#pragma clang fp contract(off)
    const int64_t n = nside;
    const double dn = (double)nside;
    const double za = fabs(z), tt = phi / (M_PI / 2);
    if (za <= 2.0 / 3.0) {
        const double t1 = dn * (0.5 + tt);
        const double t2 = dn * (z * 0.75);
        const int64_t jp = (int64_t)floor(t1 - t2), jm = (int64_t)floor(t1 + t2);
        const int64_t ir = n + 1 + jp - jm;
        const int64_t kshift = 1 - (ir & 1);
        const int64_t m4 = 4 * n;
        const int64_t ip = (((jp + jm - n + kshift + 1) >> 1) % m4 + m4) % m4;
        return 2 * n * (n - 1) + (ir - 1) * m4 + ip;
    }
    const double tp = tt - floor(tt);
    const double tmp = dn * sqrt(3.0 * (1.0 - za));
    const int64_t jp = (int64_t)floor(tp * tmp), jm = (int64_t)floor((1.0 - tp) * tmp);
    const int64_t ir = jp + jm + 1;
    const int64_t ip = ((int64_t)floor(tt * (double)ir)) % (4 * ir);
    return z > 0 ? 2 * ir * (ir - 1) + ip : 12 * n * n - 2 * ir * (ir + 1) + ip;
}

// pixel of every galaxy; inputs out of range set flag (1: position, 2: weight or ellipticity) and
// give pixel 0, so later stages stay in bounds.  With ellipticities, also the galaxy's record
// {w, w e1, w e2, w^2} (each product rounded once), so that the per-pixel pass gathers one 32-byte
// record per galaxy instead of three scattered values.
__global__ void k_ang2pix(const double *__restrict__ z, const double *__restrict__ phi,
                          const double *__restrict__ e1, const double *__restrict__ e2,
                          const double *__restrict__ w, int64_t n, int nside, uint32_t *__restrict__ pix,
                          double4 *__restrict__ rec, int *__restrict__ flag)
{
#pragma clang fp contract(off)
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        const double zz = z[j], pp = phi[j];
        int64_t p = 0;
        if (!(zz >= -1.0 && zz <= 1.0 && pp >= 0.0 && pp < 2.0 * M_PI)) {
            flag[0] = 1;
        } else {
            p = ang2pix_ring(nside, zz, pp);
        }
        if (e1) {
            const double ww = w[j], a = e1[j], b = e2[j];
            if (!(ww >= 0.0) || !isfinite(ww) || !isfinite(a) || !isfinite(b)) flag[1] = 2;
            rec[j] = make_double4(ww, ww * a, ww * b, ww * ww);
        }
        pix[j] = (uint32_t)p;
    }
}

__global__ void k_fill_i32(int32_t *__restrict__ a, int32_t *__restrict__ b, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        a[i] = 0;
        b[i] = 0;
    }
}

// [start, end) of every pixel's run in the sorted keys (empty pixels keep 0, 0)
__global__ void k_seg_bounds(const uint32_t *__restrict__ keys, int64_t n, int32_t *__restrict__ start,
                             int32_t *__restrict__ end)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t p = keys[i];
        if (i == 0 || keys[i - 1] != p) start[p] = (int32_t)i;
        if (i == n - 1 || keys[i + 1] != p) end[p] = (int32_t)(i + 1);
    }
}

// per pixel: sums over its galaxies in catalogue order, then eq. gamma_obs, Neff_pixel, noise_var,
// mask (sum w = 0: no shear; sum w^2 = 0: N_eff = 0)
__global__ void k_pix_accum(const int32_t *__restrict__ start, const int32_t *__restrict__ end,
                            const uint32_t *__restrict__ gal, const double4 *__restrict__ rec, int64_t npix, double R,
                            double se2, double n_th, double *__restrict__ g1, double *__restrict__ g2,
                            double *__restrict__ ninv, double *__restrict__ neff, uint8_t *__restrict__ mask)
{
#pragma clang fp contract(off)
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < npix; p += (int64_t)gridDim.x * blockDim.x) {
        double sw = 0.0, s1 = 0.0, s2 = 0.0, sww = 0.0;
        const int32_t b = start[p], e = end[p];
        for (int32_t i = b; i < e; ++i) {
            const double4 g = rec[gal[i]];
            sw = sw + g.x;
            s1 = s1 + g.y;
            s2 = s2 + g.z;
            sww = sww + g.w;
        }
        const double den = R * sw;
        const double ne = (sww != 0.0) ? (sw * sw) / sww : 0.0;
        g1[p] = (sw != 0.0) ? s1 / den : 0.0;
        g2[p] = (sw != 0.0) ? s2 / den : 0.0;
        neff[p] = ne;
        ninv[p] = ne / se2;
        mask[p] = ne >= n_th ? 1 : 0;
    }
}

// ================================================================================================
// Pixel ranges ("buckets" of 2^shift consecutive pixels, at most MAX_BUCKETS).  Four passes move each galaxy
// once: pixel and count per (tile, bucket); exclusive prefix over the tiles of each bucket and over the
// buckets; a stable scatter of the records {w, e1, e2, pixel in the bucket}; the sums of a bucket in LDS.
// Bound by memory, 40 bytes read and 36 written per galaxy in the scatter, 32 read in the sums, 33 written
// per pixel.  2e7 galaxies at Nside 1024: 1170 us (counts 126, prefixes 25, scatter 595, sums 426;
// the scatter's 32-byte records reach lines that no longer are in L2), against 1810 us through the sort, whose
// last pass gathered a 32-byte record per galaxy at random (870 us) after three passes over 8-byte pairs (470 us).
// 1e6 at Nside 64 246 -> 133 us, 3000 at Nside 32 61 -> 49 us.
// ================================================================================================
constexpr int MAX_BUCKETS = 4096, MAX_SHIFT = 12;
constexpr int64_t BUCKET_NPIX = (int64_t)MAX_BUCKETS << MAX_SHIFT;  // 36 bytes of LDS per pixel of a bucket
constexpr int PIX_T = 512;                                         // threads of a workgroup
constexpr int TILE_MIN = 1024, TILE_MAX = 16384;                   // galaxies of a workgroup (see pix_buckets)

// pixels of every galaxy, flag as k_ang2pix, and the tile's galaxies per bucket in hist[tile][nb]
__global__ __launch_bounds__(PIX_T) void k_pix_count(const double *__restrict__ z, const double *__restrict__ phi,
                                                     int64_t n, int tile, int nside, int shift, int nb,
                                                     uint32_t *__restrict__ pix, uint32_t *__restrict__ hist,
                                                     int *__restrict__ flag)
{
    __shared__ uint32_t h[MAX_BUCKETS];
    for (int b = threadIdx.x; b < nb; b += PIX_T) h[b] = 0;
    __syncthreads();
    const int64_t j0 = (int64_t)blockIdx.x * tile, j1 = j0 + tile < n ? j0 + tile : n;
    for (int64_t j = j0 + threadIdx.x; j < j1; j += PIX_T) {
        const double zz = z[j], pp = phi[j];
        uint32_t p = 0;
        if (!(zz >= -1.0 && zz <= 1.0 && pp >= 0.0 && pp < 2.0 * M_PI)) flag[0] = 1;
        else p = (uint32_t)ang2pix_ring(nside, zz, pp);
        pix[j] = p;
        atomicAdd(&h[p >> shift], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += PIX_T) hist[(int64_t)blockIdx.x * nb + b] = h[b];
}

// every column of hist[ntiles][nb] to its exclusive prefix; the column sums to total.  32 columns a
// workgroup, their rows in 32 parts.
__global__ __launch_bounds__(1024) void k_pix_colscan(uint32_t *__restrict__ hist, int ntiles, int nb,
                                                      uint32_t *__restrict__ total)
{
    __shared__ uint32_t s[32][33];
    const int c = blockIdx.x * 32 + (threadIdx.x & 31), part = threadIdx.x >> 5;
    const int per = (ntiles + 31) / 32, t0 = part * per, t1 = t0 + per < ntiles ? t0 + per : ntiles;
    uint32_t sum = 0;
    if (c < nb)
        for (int t = t0; t < t1; ++t) sum += hist[(int64_t)t * nb + c];
    s[part][threadIdx.x & 31] = sum;
    __syncthreads();
    if (c >= nb) return;
    uint32_t run = 0;
    for (int q = 0; q < part; ++q) run += s[q][threadIdx.x & 31];
    if (part == 31) total[c] = run + sum;
    for (int t = t0; t < t1; ++t) {
        const uint32_t v = hist[(int64_t)t * nb + c];
        hist[(int64_t)t * nb + c] = run;
        run += v;
    }
}

// first record of every bucket, and n at start[nb] (one workgroup)
__global__ __launch_bounds__(1024) void k_pix_starts(const uint32_t *__restrict__ total, int nb,
                                                     uint32_t *__restrict__ start)
{
    constexpr int PER = MAX_BUCKETS / 1024;
    __shared__ uint32_t s[1024];
    const int b0 = threadIdx.x * PER;
    uint32_t sum = 0;
    for (int q = 0; q < PER; ++q) sum += b0 + q < nb ? total[b0 + q] : 0u;
    s[threadIdx.x] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const uint32_t v = (int)threadIdx.x >= d ? s[threadIdx.x - d] : 0u;
        __syncthreads();
        s[threadIdx.x] += v;
        __syncthreads();
    }
    uint32_t run = s[threadIdx.x] - sum;
    for (int q = 0; q < PER; ++q) {
        if (b0 + q <= nb) start[b0 + q] = run;
        if (b0 + q < nb) run += total[b0 + q];
    }
    if (threadIdx.x == 1023 && nb == MAX_BUCKETS) start[nb] = run;
}

// lanes of one wave hand LDS values to each other (its LDS accesses execute in order)
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// the tile's records to their buckets in catalogue order.  Each wave takes an eighth of the tile, 64 galaxies
// at a time: it counts them per bucket first, and with the counts of the waves before it a galaxy's place is
// the bucket's first free one plus the lanes before it with the same bucket (found bit by bit by ballots).
__global__ __launch_bounds__(PIX_T) void k_pix_scatter(const uint32_t *__restrict__ pix, const double *__restrict__ e1,
                                                       const double *__restrict__ e2, const double *__restrict__ w,
                                                       int64_t n, int tile, int shift, int nb, int bits,
                                                       const uint32_t *__restrict__ hist,
                                                       const uint32_t *__restrict__ start, double4 *__restrict__ rec,
                                                       int *__restrict__ flag)
{
    constexpr int W = PIX_T / 64;
    __shared__ uint32_t first[MAX_BUCKETS];
    __shared__ uint32_t cnt2[W][MAX_BUCKETS / 2];  // two 16-bit counts (at most TILE_MAX) a word
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint16_t *cnt = reinterpret_cast<uint16_t *>(cnt2[wave]);
    for (int b = threadIdx.x; b < nb; b += PIX_T) first[b] = start[b] + hist[(int64_t)blockIdx.x * nb + b];
    for (int b = lane; b < (nb + 1) / 2; b += 64) cnt2[wave][b] = 0;
    __syncthreads();
    const int part = tile / W;  // galaxies of a wave
    const int64_t j0 = (int64_t)blockIdx.x * tile + (int64_t)wave * part, j1 = j0 + part < n ? j0 + part : n;
    for (int64_t j = j0 + lane; j < j1; j += 64) {
        const uint32_t b = pix[j] >> shift;
        atomicAdd(&cnt2[wave][b >> 1], (b & 1) ? 0x10000u : 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += PIX_T) {
        uint32_t run = 0;
#pragma unroll
        for (int v = 0; v < W; ++v) {
            uint16_t *c = reinterpret_cast<uint16_t *>(cnt2[v]) + b;
            const uint32_t t = *c;
            *c = (uint16_t)run;
            run += t;
        }
    }
    __syncthreads();
    struct In {
        uint32_t p;
        double w, a, b;
    };
    auto load = [&](int64_t j) {
        In v = {0, 0.0, 0.0, 0.0};
        if (j < j1) v = In{pix[j], w[j], e1[j], e2[j]};
        return v;
    };
    // four times 64 galaxies on their way while four times 64 are placed (loads and stores are waited for in
    // one order, so the loads of each 64 would also wait for the stores of the 64 before)
    constexpr int U = 4;
    In v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = load(j0 + 64 * u + lane);
    for (int64_t jb = j0; jb < j1; jb += 64 * U) {
        In nx[U];
#pragma unroll
        for (int u = 0; u < U; ++u) nx[u] = load(jb + 64 * (U + u) + lane);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = jb + 64 * u + lane < j1;
            const uint32_t b = v[u].p >> shift;
            uint64_t same = __ballot(on);
            for (int q = 0; q < bits; ++q) {
                const bool bit = (b >> q) & 1;
                const uint64_t t = __ballot(bit);
                same &= bit ? t : ~t;
            }
            const int before = __popcll(same & ((1ull << lane) - 1)), all = __popcll(same);
            if (on) {
                if (!(v[u].w >= 0.0) || !isfinite(v[u].w) || !isfinite(v[u].a) || !isfinite(v[u].b)) flag[1] = 2;
                const uint32_t c = cnt[b];
                rec[(int64_t)first[b] + c + before] = make_double4(
                    v[u].w, v[u].a, v[u].b, __longlong_as_double((long long)(v[u].p & ((1u << shift) - 1))));
                wave_lds_fence();
                if (before == all - 1) cnt[b] = (uint16_t)(c + all);
            }
            wave_lds_fence();
        }
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = nx[u];
    }
}

constexpr int PIX_Q = 2;  // records of a thread per batch
// Sums and outputs of one bucket.  The workgroup takes its records PIX_Q PIX_B at a time; in each turn the first
// pending record of every pixel (the largest of turn * PIX_Q PIX_B + its distance from the end) adds to the
// pixel's sums, until none is left.  Workgroups stay for several buckets and load the next one's records
// before they write a bucket's outputs (up to 144 KB of LDS leave one workgroup on a compute unit, with no
// other to fill its waits).  Nothing is written when an input was out of range (flag).
// A batch takes as many turns as its fullest pixel has records: 17 of 512 records over 64 pixels, 45 over 16.  So a
// bucket of at most PIX_DENSE pixels with more than four records for each is sorted by pixel in LDS batch by batch
// (stable, as in the scatter), and four threads per pixel add its run, one for each sum.  2e7 galaxies in 0.1 of
// the sky, us: Nside 128 2190 -> 1390, Nside 64 4740 -> 1680, Nside 16 42700 -> 14400 (through the radix sort 1960, 4440, 58200).
constexpr int PIX_DENSE = 64;
constexpr int pix_lds(int shift)
{
    // four sums and a tag per pixel; dense buckets: the sorted batch, counts of its eight groups of 64, run bounds
    return (36 << shift) + ((1 << shift) <= PIX_DENSE ? 24 * PIX_Q * 256 + 4 * ((PIX_Q * 4 + 1) << shift) + 4 : 0);
}
template <int PIX_B>
__global__ __launch_bounds__(PIX_B) void k_pix_bucket(const uint32_t *__restrict__ start,
                                                      const double4 *__restrict__ rec, int shift, int nb,
                                                      int64_t npix, double R, double se2, double n_th, double *__restrict__ g1,
                                                      double *__restrict__ g2, double *__restrict__ ninv,
                                                      double *__restrict__ neff, uint8_t *__restrict__ mask,
                                                      const int *__restrict__ flag)
{
#pragma clang fp contract(off)
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ int more[2];
    const int np = 1 << shift;
    constexpr int BATCH = PIX_Q * PIX_B, WAVES = PIX_B / 64, GROUPS = PIX_Q * WAVES;
    const bool few = PIX_B == 256 && np <= PIX_DENSE;    // (the dense buffers are there)
    double *sum = reinterpret_cast<double *>(smem_raw);  // sum w, w e1, w e2, w^2, np of each
    double *stage = sum + 4 * np;                        // w, e1, e2 of a batch by pixel, BATCH of each
    uint32_t *tag = reinterpret_cast<uint32_t *>(stage + (few ? 3 * BATCH : 0));
    uint32_t *cnt = tag + np, *run = cnt + GROUPS * np;  // [group][pixel] counts, np + 1 run bounds
    if (flag[0] || flag[1]) return;
    for (int i = threadIdx.x; i < 4 * np; i += PIX_B) sum[i] = 0.0;
    for (int i = threadIdx.x; i < np; i += PIX_B) tag[i] = 0;
    if (threadIdx.x == 0) more[0] = more[1] = 0;
    __syncthreads();
    constexpr uint32_t TURNS = 0xffffffffu / BATCH - 1;
    const double4 none = make_double4(0.0, 0.0, 0.0, 0.0);
    double4 v[PIX_Q];
    auto first = [&](int64_t a, int64_t e) {
#pragma unroll
        for (int q = 0; q < PIX_Q; ++q) {
            const int64_t i = a + q * PIX_B + threadIdx.x;
            v[q] = i < e ? rec[i] : none;
        }
    };
    uint32_t turn = 0;
    int bk = blockIdx.x;
    int64_t b0 = start[bk], b1 = start[bk + 1];
    first(b0, b1);
    while (true) {
        const int bn = bk + (int)gridDim.x;
        const int64_t n0 = bn < nb ? start[bn] : 0, n1 = bn < nb ? start[bn + 1] : 0;
        const bool dense = few && b1 - b0 > 4 * np;
        double mine = 0.0;  // dense: sum (threadIdx.x & 3) of pixel threadIdx.x / 4
        for (int64_t b = b0; b < b1; b += BATCH) {
            double4 nx[PIX_Q];
            bool pend[PIX_Q];
            int px[PIX_Q];
#pragma unroll
            for (int q = 0; q < PIX_Q; ++q) {
                const int64_t i = b + q * PIX_B + threadIdx.x;
                pend[q] = i < b1;
                px[q] = (int)__double_as_longlong(v[q].w);
                nx[q] = i + BATCH < b1 ? rec[i + BATCH] : none;
            }
            if (dense) {
                const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
                for (int i = threadIdx.x; i < GROUPS * np; i += PIX_B) cnt[i] = 0;
                __syncthreads();
                int before[PIX_Q];
#pragma unroll
                for (int q = 0; q < PIX_Q; ++q) {
                    uint64_t same = __ballot(pend[q]);
                    for (int k = 0; k < shift; ++k) {
                        const bool bit = (px[q] >> k) & 1;
                        const uint64_t t = __ballot(bit);
                        same &= bit ? t : ~t;
                    }
                    before[q] = __popcll(same & ((1ull << lane) - 1));
                    if (pend[q] && before[q] == 0) cnt[(q * WAVES + wave) * np + px[q]] = __popcll(same);
                }
                __syncthreads();
                if (wave == 0) {
                    uint32_t all = 0;
                    if (lane < np)
                        for (int g = 0; g < GROUPS; ++g) {
                            const uint32_t c = cnt[g * np + lane];
                            cnt[g * np + lane] = all;
                            all += c;
                        }
                    uint32_t upto = all;
                    for (int d = 1; d < 64; d <<= 1) {
                        const uint32_t u = __shfl_up(upto, d, 64);
                        if (lane >= d) upto += u;
                    }
                    if (lane < np) run[lane + 1] = upto;
                    if (lane == 0) run[0] = 0;
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < PIX_Q; ++q)
                    if (pend[q]) {
                        const int at = (int)(run[px[q]] + cnt[(q * WAVES + wave) * np + px[q]]) + before[q];
                        stage[at] = v[q].x;
                        stage[BATCH + at] = v[q].y;
                        stage[2 * BATCH + at] = v[q].z;
                    }
                __syncthreads();
                const int p = threadIdx.x >> 2, c = threadIdx.x & 3;
                if (p < np) {
                    const int e = (int)run[p + 1];
#pragma unroll 4
                    for (int i = (int)run[p]; i < e; ++i) {
                        const double ww = stage[i], o = c == 1 ? stage[BATCH + i] : c == 2 ? stage[2 * BATCH + i] : ww;
                        mine = mine + (c ? ww * o : ww);
                    }
                }
#pragma unroll
                for (int q = 0; q < PIX_Q; ++q) v[q] = nx[q];
                continue;
            }
            for (bool again = true; again;) {
                if (++turn == TURNS) {  // the turn count of the tags starts over
                    for (int i = threadIdx.x; i < np; i += PIX_B) tag[i] = 0;
                    turn = 1;
                    __syncthreads();
                }
                uint32_t key[PIX_Q];
#pragma unroll
                for (int q = 0; q < PIX_Q; ++q) {
                    key[q] = turn * BATCH + (BATCH - 1 - (q * PIX_B + threadIdx.x));
                    if (pend[q]) atomicMax(&tag[px[q]], key[q]);
                }
                __syncthreads();
                bool left = false;
#pragma unroll
                for (int q = 0; q < PIX_Q; ++q) {
                    if (pend[q] && tag[px[q]] == key[q]) {
                        const double ww = v[q].x;
                        const int i = px[q];
                        sum[i] = sum[i] + ww;
                        sum[np + i] = sum[np + i] + ww * v[q].y;
                        sum[2 * np + i] = sum[2 * np + i] + ww * v[q].z;
                        sum[3 * np + i] = sum[3 * np + i] + ww * ww;
                        pend[q] = false;
                    }
                    left |= pend[q];
                }
                if (left) more[turn & 1] = 1;
                if (threadIdx.x == 0) more[(turn + 1) & 1] = 0;
                __syncthreads();
                again = more[turn & 1] != 0;
            }
#pragma unroll
            for (int q = 0; q < PIX_Q; ++q) v[q] = nx[q];
        }
        if (bn < nb) first(n0, n1);
        if (dense) {
            if ((int)threadIdx.x < 4 * np) sum[(threadIdx.x & 3) * np + (threadIdx.x >> 2)] = mine;
            __syncthreads();
        }
        for (int i = threadIdx.x; i < np; i += PIX_B) {
            const int64_t p = ((int64_t)bk << shift) + i;
            const double sw = sum[i], s1 = sum[np + i], s2 = sum[2 * np + i], sww = sum[3 * np + i];
            sum[i] = sum[np + i] = sum[2 * np + i] = sum[3 * np + i] = 0.0;
            if (p >= npix) break;
            const double den = R * sw;
            const double ne = (sww != 0.0) ? (sw * sw) / sww : 0.0;
            g1[p] = (sw != 0.0) ? s1 / den : 0.0;
            g2[p] = (sw != 0.0) ? s2 / den : 0.0;
            neff[p] = ne;
            ninv[p] = ne / se2;
            mask[p] = ne >= n_th ? 1 : 0;
        }
        if (bn >= nb) break;
        bk = bn;
        b0 = n0;
        b1 = n1;
        __syncthreads();
    }
}

static int key_bits(int64_t npix)
{
    int b = 1;
    while (((int64_t)1 << b) < npix) ++b;
    return b;
}

static int grid_for(int64_t n)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 16384));
}

// workspace: galaxy records, unsorted keys, sorted keys, sorted galaxy indices, pixel runs,
// radix-sort storage
struct PixWork {
    double4 *rec;
    uint32_t *keys, *keys_s, *gal_s;
    int32_t *seg_a, *seg_b;
    void *tmp;
    size_t tmp_bytes;
};

static int64_t a256(int64_t b) { return (b + 255) / 256 * 256; }

static hipError_t pixelize_work(Plan &P, int64_t n_gal, void *base, int64_t *bytes, PixWork *pw)
{
    size_t tb = 0;
    const uint32_t *kin = nullptr;
    uint32_t *kout = nullptr, *vout = nullptr;
    hipError_t e = rocprim::radix_sort_pairs(nullptr, tb, kin, kout, rocprim::counting_iterator<uint32_t>(0u), vout,
                                             (size_t)std::max<int64_t>(n_gal, 1), 0u, (unsigned)key_bits(P.npix),
                                             P.stream);
    if (e != hipSuccess) return e;
    const int64_t ng = std::max<int64_t>(n_gal, 1);
    const int64_t total = a256(32 * ng) + 3 * a256(4 * ng) + 2 * a256(4 * P.npix) + a256((int64_t)tb);
    if (bytes) *bytes = total;
    if (pw && base) {
        char *c = (char *)base;
        pw->rec = (double4 *)c;
        c += a256(32 * ng);
        pw->keys = (uint32_t *)c;
        c += a256(4 * ng);
        pw->keys_s = (uint32_t *)c;
        c += a256(4 * ng);
        pw->gal_s = (uint32_t *)c;
        c += a256(4 * ng);
        pw->seg_a = (int32_t *)c;
        c += a256(4 * P.npix);
        pw->seg_b = (int32_t *)c;
        c += a256(4 * P.npix);
        pw->tmp = c;
        pw->tmp_bytes = tb;
    }
    return hipSuccess;
}

// the bucket path: pixels per bucket the smallest power of two, at least 16 (a wave's worth of adds per turn
// and few galaxies left over), that gives at most MAX_BUCKETS
struct PixBuckets {
    int shift = 4, nb, bits = 0, tile = TILE_MAX, ntiles;
    double4 *rec;
    uint32_t *pix, *hist, *total, *start;
    int64_t bytes;
};
static PixBuckets pix_buckets(Plan &P, int64_t n, void *base)
{
    PixBuckets B;
    while (((P.npix - 1) >> B.shift) >= MAX_BUCKETS) ++B.shift;
    B.nb = (int)((P.npix - 1) >> B.shift) + 1;
    while ((1 << B.bits) < B.nb) ++B.bits;
    const int64_t ng = std::max<int64_t>(n, 1);
    // long tiles give long runs per bucket; down to TILE_MIN as long as there are fewer than four for each CU
    while (B.tile > TILE_MIN && ng < (int64_t)1024 * B.tile) B.tile /= 2;
    B.ntiles = (int)((ng + B.tile - 1) / B.tile);
    char *c = (char *)base;
    auto take = [&](int64_t bytes) {
        char *q = c;
        c += a256(bytes);
        return q;
    };
    B.rec = (double4 *)take(32 * ng);
    B.pix = (uint32_t *)take(4 * ng);
    B.hist = (uint32_t *)take((int64_t)4 * B.nb * B.ntiles);
    B.total = (uint32_t *)take((int64_t)4 * B.nb);
    B.start = (uint32_t *)take((int64_t)4 * (B.nb + 1));
    B.bytes = c - (char *)base;
    return B;
}

// more pixels than BUCKET_NPIX (Nside > 1182) would need more buckets, or more LDS per bucket, than there is
bool pixelize_in_buckets(const Plan &P) { return P.npix <= BUCKET_NPIX; }

hipError_t launch_pixelize_buckets(Plan &P, const double *z, const double *phi, const double *e1, const double *e2,
                                   const double *w, int64_t n, double R, double se2, double n_th, void *work,
                                   double *g1, double *g2, double *ninv, double *neff, uint8_t *mask)
{
    const PixBuckets B = pix_buckets(P, n, work);
    const size_t sm = pix_lds(B.shift);
    int cus = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, P.dev);
    if (e != hipSuccess) return e;
    k_pix_count<<<B.ntiles, PIX_T, 0, P.stream>>>(z, phi, n, B.tile, P.nside, B.shift, B.nb, B.pix, B.hist,
                                                  P.d_cmp_flag);
    k_pix_colscan<<<(B.nb + 31) / 32, 1024, 0, P.stream>>>(B.hist, B.ntiles, B.nb, B.total);
    k_pix_starts<<<1, 1024, 0, P.stream>>>(B.total, B.nb, B.start);
    k_pix_scatter<<<B.ntiles, PIX_T, 0, P.stream>>>(B.pix, e1, e2, w, n, B.tile, B.shift, B.nb, B.bits, B.hist, B.start,
                                                    B.rec, P.d_cmp_flag);
    // as many workgroups as stay on the device together: eight of 256 threads a compute unit, for buckets of up to
    // 512 pixels (18 KB of LDS), or one or two of 1024
    auto sums = [&](auto kern, int threads, int blocks) {
        e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
        if (e != hipSuccess) return;
        kern<<<std::min(B.nb, cus * blocks), threads, sm, P.stream>>>(B.start, B.rec, B.shift, B.nb, P.npix, R, se2, n_th,
                                                                      g1, g2, ninv, neff, mask, P.d_cmp_flag);
    };
    if (B.shift <= 9) sums(k_pix_bucket<256>, 256, 8);
    else sums(k_pix_bucket<1024>, 1024, B.shift <= 10 ? 2 : 1);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

void launch_ang2pix(Plan &P, const double *z, const double *phi, const double *e1, const double *e2, const double *w,
                    int64_t n, uint32_t *pix, double4 *rec)
{
    if (n > 0) k_ang2pix<<<grid_for(n), 256, 0, P.stream>>>(z, phi, e1, e2, w, n, P.nside, pix, rec, P.d_cmp_flag);
}

hipError_t launch_pixelize(Plan &P, int64_t n, double R, double se2, double n_th, void *work, double *g1, double *g2,
                           double *ninv, double *neff, uint8_t *mask)
{
    PixWork pw;
    int64_t total = 0;
    hipError_t e = pixelize_work(P, n, work, &total, &pw);
    if (e != hipSuccess) return e;
    k_fill_i32<<<grid_for(P.npix), 256, 0, P.stream>>>(pw.seg_a, pw.seg_b, P.npix);
    if (n > 0) {
        size_t tb = pw.tmp_bytes;
        e = rocprim::radix_sort_pairs(pw.tmp, tb, pw.keys, pw.keys_s, rocprim::counting_iterator<uint32_t>(0u),
                                      pw.gal_s, (size_t)n, 0u, (unsigned)key_bits(P.npix), P.stream);
        if (e != hipSuccess) return e;
        k_seg_bounds<<<grid_for(n), 256, 0, P.stream>>>(pw.keys_s, n, pw.seg_a, pw.seg_b);
    }
    k_pix_accum<<<grid_for(P.npix), 256, 0, P.stream>>>(pw.seg_a, pw.seg_b, pw.gal_s, pw.rec, P.npix, R, se2, n_th, g1,
                                                        g2, ninv, neff, mask);
    return hipGetLastError();
}

hipError_t pixelize_work_bytes(Plan &P, int64_t n_gal, int64_t *bytes)
{
    if (pixelize_in_buckets(P)) {
        *bytes = pix_buckets(P, n_gal, nullptr).bytes;
        return hipSuccess;
    }
    return pixelize_work(P, n_gal, nullptr, bytes, nullptr);
}

uint32_t *pixelize_keys(Plan &P, int64_t n, void *work, double4 **rec)
{
    PixWork pw;
    if (pixelize_work(P, n, work, nullptr, &pw) != hipSuccess) return nullptr;
    *rec = pw.rec;
    return pw.keys;
}

}  // namespace akra
