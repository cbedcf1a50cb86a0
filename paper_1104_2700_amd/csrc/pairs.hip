// Full FP64 sweeps by pairs: every particle of every system is active, so
// each pair (i, j) is evaluated once and its terms go to both particles.
//
// The one-sided sweep issues 33 FP64 instructions and one v_rsq_f64 per
// interaction.  A pair takes 24 shared ones (differences, r^2, 1/sqrt, r.v,
// v - b r), the v_rsq_f64 and 8 for each side: 20 and half a v_rsq_f64 per
// interaction, 88 cycles of a SIMD against 148.  Both sweeps are bound by
// FP64 issue at the clock that the chip holds under it (about 2.0 GHz), so
// the count is the time.  Measured (MI355X, default shapes, whole calls,
// one-sided / by pairs): N = 65536 4.95 / 3.17 ms, N = 9973 129 / 112 us, 256
// clusters of 263 ... 8080 particles 4.68 / 2.18 ms; potentials alone (the
// energy sweep) N = 50021 1.50 / 0.77 ms.
//
// Layout.  A workgroup of W waves holds an i-block of 64 K W particles in
// registers (K per lane, with their seven sums) and streams j tiles of 64 W
// particles through LDS.  Within a tile a wave takes 64 of the j at a time:
// in step s lane l meets j = (l + s) mod 64, so the lanes of a wave always
// hold different j and add the j-side terms (of their K particles, summed in
// registers first) to the tile's sums with LDS adds that never meet; the
// waves of the workgroup take the tile's 64-particle parts in turn, a
// barrier between turns.  Every sum is therefore taken in a fixed order.
// K = 4 keeps the 7 LDS reads and 7 LDS adds of a step (28 and 56 cycles of
// the unit's LDS) well under its 4 x 176 FP64 cycles; moving j and its sums
// between lanes by DPP would add 28 moves of four cycles to a step.  Four
// particles a lane take up to 241 registers: two waves a SIMD.  (Reading the next
// step's j or the next tile ahead, and LDS read-modify-write in place of the
// adds, measured the same or 3 % slower.)
//
// Which pairs.  With nb i-blocks in a system, block a meets itself (one-sided,
// the self pair masked by index) and the blocks a + 1 ... a + (nb - 1) / 2
// (mod nb); for even nb also a + nb / 2 when a < nb / 2.  Every pair of
// blocks is met once and all rows have the same length.  A row's j tiles are
// cut into chunks (PairShape::lev); a work item is (block, chunk).
//
// Partial sums.  An item writes its i-side sums to slot `chunk` and every j
// tile's sums to slot nch + d - 1, d the distance of the tile's block from
// the item's: each particle has one value per chunk of its own row and one
// per block that met it.  pair_reduce_kernel adds them in a fixed order.
#include "hermite_internal.h"
#include "pair.h"
#include "plan.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace hm {
namespace {

// Blocks of a system of nc particles and the j tiles of block a's row.
__host__ __device__ inline int pair_blocks(int64_t nc, int bi)
{
    return (int)((nc + bi - 1) / bi);
}

__host__ __device__ inline int pair_row(int nb, int a, int k)
{
    const int half = (nb & 1) == 0 && a < nb / 2 ? 1 : 0;
    return k * (1 + (nb - 1) / 2 + half);
}

// Chunks of a row of u tiles.
__host__ __device__ inline int pair_chunks(const PairShape& sh, int u)
{
    int c = 0;
    while (c < sh.nch && sh.lev[c] < u) ++c;
    return c;
}

// Particles past a block's end: massless, far away and apart from each
// other, so that a pair with one adds exactly zero.
constexpr double kPadI = 2.0e30, kPadJ = 1.0e30;

// Where the pair sweep runs, and in which shape.
// One system from 6000 particles on (potentials: 4500): below, the pair
// tiles are too few to fill the chip (fresh contexts, one-sided / by pairs:
// 4000 38 / 41 us, 6001 70 / 66, 8000 102 / 90, 12000 226 / 163; energy 4000
// 29 / 29, 6001 45 / 40).
constexpr int64_t kPairMin = 6000, kPairMinPot = 4500;
// Particles a lane and waves a workgroup: small systems take small items
// (K = 3, one wave: 14001 particles 186 us, with K = 4 205), larger ones
// K = 4 (32768: 870 us, with K = 3 886), and from 45000 on (potentials:
// 24576) four waves share a tile: half the j-side partial sums of one-wave
// blocks (65536: 3.24 against 3.35 ms; 40000: 1.32 against 1.29).
constexpr int64_t kPairFour = 20000;
constexpr int64_t kPairWide = 45000, kPairWidePot = 24576;
constexpr int64_t kPairMaxN = (int64_t)1 << 23;   // rows of at most 2^15 - 1 tiles
// Ensembles whose largest cluster fits 43 blocks (17 chunks and 21 block
// slots of partial sums), with at least 6e7 interactions (n^2 / C, a lower
// bound; 4e7 from 30 clusters on, which fill the last round more evenly) and
// clusters of 256 particles on average (1500 of 30 ... 300: 105 one-sided,
// 128 by pairs, whose blocks of 192 are half empty).  One-sided / by pairs:
// 20 clusters of 600 ... 2500, 3.5e7, 76 / 94 us; 7 of 600 ... 8192, 5.8e7,
// 133 / 164; 20 of 600 ... 4000, 6.4e7, 143 / 132; 10 of 600 ... 8192, 8.4e7,
// 241 / 171; 30 of 64 ... 5500, 4.5e7, 181 / 136.
constexpr int64_t kPairMaxCluster = 8192, kPairMeanCluster = 256;
constexpr double kPairEnsemble = 6.0e7, kPairManyEnsemble = 4.0e7;
constexpr int kPairMany = 30;
constexpr int kPairClusterSlots = 17;

// Two levels of sums, as in the one-sided sweep: a register adds a run of at
// most 256 terms, and the runs are added up by themselves.  Workgroups of
// K = 4 have long chunks (2816 terms at N = 65536): each tile's sums go to a
// second sum, in LDS.  Those of K = 3 have no LDS to spare (16 KB instead of 7
// leave 9 workgroups a unit for 12: N = 9973 110 -> 124 us), so their chunks
// end after four tiles of 64.  (Root mean square error of the acceleration,
// one-sided / by pairs in one level / in two: N = 65536 1.47 / 2.25 / 1.40e-16,
// 100000 1.42 / 3.22 / 1.36e-16, 44000 1.62 / 2.13 / 1.44e-16; times as with
// one level: 65536 3.20 / 3.19 ms, 9973 113.9 / 114.8 us.)
constexpr int kPairRun = 4;
__host__ __device__ constexpr bool pair_two_levels(int k, bool pot_only)
{
    return pot_only || k > 3;
}

// One particle of the sweep: coordinates (velocities), mass, sums.
template <bool POT>
struct PairI {
    static constexpr int NC = POT ? 3 : 6;   // coordinates
    static constexpr int NS = POT ? 1 : 7;   // sums: acc, jerk, m/r
    double c[NC], m, s[NS];
};

// The terms of a pair that both particles share: differences d (r, then v;
// v becomes v - 3 (r.v)/s r), 1/sqrt(s) and 1/s^{3/2}.
template <bool POT>
__device__ __forceinline__ void pair_shared(const double (&cj)[PairI<POT>::NC],
                                            const double (&ci)[PairI<POT>::NC], double eps2,
                                            double (&d)[PairI<POT>::NC], double& ri)
{
#pragma unroll
    for (int q = 0; q < PairI<POT>::NC; ++q) d[q] = cj[q] - ci[q];
    const double r2 = fma(d[0], d[0], fma(d[1], d[1], fma(d[2], d[2], eps2)));
    ri = rsqrt_f64(r2);
}

template <bool POT>
__device__ __forceinline__ void pair_finish(double (&d)[PairI<POT>::NC], double ri, double& ri3)
{
    if constexpr (!POT) {
        const double ri2 = ri * ri;
        ri3 = ri * ri2;
        const double rv = fma(d[0], d[3], fma(d[1], d[4], d[2] * d[5]));
        const double b3 = (rv * ri2) * 3.0;
#pragma unroll
        for (int q = 0; q < 3; ++q) d[3 + q] = fma(-b3, d[q], d[3 + q]);
    }
}

template <bool POT>
__device__ __forceinline__ void pair_side(double m, const double (&d)[PairI<POT>::NC], double ri,
                                          double ri3, double (&s)[PairI<POT>::NS])
{
    if constexpr (!POT) {
        const double m3 = m * ri3;
#pragma unroll
        for (int q = 0; q < 6; ++q) s[q] = fma(m3, d[q], s[q]);
    }
    s[PairI<POT>::NS - 1] = fma(m, ri, s[PairI<POT>::NS - 1]);
}

template <int K, int W, bool POT>
__global__ void __launch_bounds__(64 * W, 2)
pair_sweep_kernel(SweepArgs a, PairShape sh, uint32_t* queue)
{
    constexpr int kBI = 64 * K * W, kJT = 64 * W;
    constexpr int NC = PairI<POT>::NC, NS = PairI<POT>::NS;
    __shared__ double jc[NC + 1][kJT];   // coordinates and mass of the tile
    __shared__ double js[NS][kJT];       // its sums
    // the i-side sums' second level, a lane its own: acc and jerk here, the
    // potential in a register (seven rows leave no room for a second workgroup)
    constexpr bool kTop = pair_two_levels(K, POT), kTopLds = kTop && !POT;
    __shared__ double s_top[kTopLds ? NS - 1 : 1][kTopLds ? kBI : 1];
    __shared__ int32_t s_item;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t n = a.n;
    const bool many = a.n_clusters > 1;
    const int total = many ? a.plan->total_items : sh.items;

    for (int item = blockIdx.x; item < total;) {
        // ---- the item: cluster c, block ab, chunk ch ------------------------
        int64_t cb = 0, ce = n;
        int ab, ch, nb;
        double eps2 = a.eps2_c ? a.eps2_c[0] : a.eps2;   // one system, or one cluster
        if (many) {
            const int c = upper_bound_i32(a.item_off, a.n_clusters + 1, item) - 1;
            cb = a.offsets[c];
            ce = a.offsets[c + 1];
            eps2 = a.eps2_c[c];
            nb = pair_blocks(ce - cb, kBI);
            const int local = item - a.item_off[c];
            ch = local / nb;
            ab = local - ch * nb;
        } else {
            nb = pair_blocks(n, kBI);
            ch = item / nb;
            ab = item - ch * nb;
        }
        const int row = pair_row(nb, ab, K);
        const int u0 = sh.lev[ch];
        const int u1 = row < sh.lev[ch + 1] ? row : sh.lev[ch + 1];
        if (u0 < u1) {
            const int64_t ib = cb + (int64_t)ab * kBI;
            const int icnt = (int)(ce - ib < kBI ? ce - ib : kBI);
            const bool busy = wave * K * 64 < icnt;   // this wave holds a particle
            double ci[K][NC], mi[K], si[K][NS], top[K];
#pragma unroll
            for (int q = 0; q < K; ++q) {
                const int k = (wave * K + q) * 64 + lane;
                const bool ok = k < icnt;
                const int64_t g = ib + (ok ? k : 0);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    ci[q][d] = ok ? a.xp[d * n + g] : kPadI;
                    if constexpr (!POT) ci[q][3 + d] = ok ? a.vp[d * n + g] : 0.0;
                }
                mi[q] = ok ? a.m[g] : 0.0;
#pragma unroll
                for (int r = 0; r < NS; ++r) si[q][r] = 0.0;
                top[q] = 0.0;
                if constexpr (kTopLds) {
#pragma unroll
                    for (int r = 0; r < NS - 1; ++r) s_top[r][k] = 0.0;
                }
            }
            for (int u = u0; u < u1; ++u) {
                const int dist = u / K, t = u - dist * K;
                int bb = ab + dist;
                if (bb >= nb) bb -= nb;
                const int64_t jb = cb + (int64_t)bb * kBI + t * kJT;
                if (jb >= ce) continue;
                const int cnt = (int)(ce - jb < kJT ? ce - jb : kJT);
                __syncthreads();   // the tile before is read (and written out)
                {
                    const bool ok = tid < cnt;
                    const int64_t g = jb + (ok ? tid : 0);
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        jc[d][tid] = ok ? a.xp[d * n + g] : kPadJ;
                        if constexpr (!POT) jc[3 + d][tid] = ok ? a.vp[d * n + g] : 0.0;
                    }
                    jc[NC][tid] = ok ? a.m[g] : 0.0;
#pragma unroll
                    for (int r = 0; r < NS; ++r) js[r][tid] = 0.0;
                }
                __syncthreads();
                if (dist == 0) {
                    // the block with itself: the i side only
                    if (busy) {
                        for (int p = 0; p < cnt; ++p) {
                            double cj[NC];
#pragma unroll
                            for (int d = 0; d < NC; ++d) cj[d] = jc[d][p];
                            const double mj = jc[NC][p];
#pragma unroll
                            for (int q = 0; q < K; ++q) {
                                double d[NC], ri, ri3 = 0.0;
                                pair_shared<POT>(cj, ci[q], eps2, d, ri);
                                ri = t * kJT + p == (wave * K + q) * 64 + lane ? 0.0 : ri;
                                pair_finish<POT>(d, ri, ri3);
                                pair_side<POT>(mj, d, ri, ri3, si[q]);
                            }
                        }
                    }
                } else {
                    for (int ph = 0; ph < W; ++ph) {
                        const int sub = (wave + ph) % W;
                        if (busy && sub * 64 < cnt) {
                            for (int s = 0; s < 64; ++s) {
                                const int p = sub * 64 + ((lane + s) & 63);
                                double cj[NC], sj[NS];
#pragma unroll
                                for (int d = 0; d < NC; ++d) cj[d] = jc[d][p];
                                const double mj = jc[NC][p];
#pragma unroll
                                for (int r = 0; r < NS; ++r) sj[r] = 0.0;
#pragma unroll
                                for (int q = 0; q < K; ++q) {
                                    double d[NC], ri, ri3 = 0.0;
                                    pair_shared<POT>(cj, ci[q], eps2, d, ri);
                                    pair_finish<POT>(d, ri, ri3);
                                    pair_side<POT>(mj, d, ri, ri3, si[q]);
                                    pair_side<POT>(mi[q], d, ri, ri3, sj);
                                }
#pragma unroll
                                for (int r = 0; r < NS; ++r) unsafeAtomicAdd(&js[r][p], sj[r]);
                            }
                        }
                        __syncthreads();   // the next wave's turn at this part
                    }
                    if (tid < cnt) {
                        // the j side saw -r and -v: acc and jerk change sign, as
                        // the potential -m/r does
                        double* dst = a.partial + (int64_t)(sh.nch + dist - 1) * NS * n + jb + tid;
#pragma unroll
                        for (int r = 0; r < NS; ++r) dst[(int64_t)r * n] = -js[r][tid];
                    }
                }
                if constexpr (kTop) {   // the tile's sums to the second level
#pragma unroll
                    for (int q = 0; q < K; ++q) {
                        if constexpr (kTopLds) {
#pragma unroll
                            for (int r = 0; r < NS - 1; ++r) {
                                s_top[r][(wave * K + q) * 64 + lane] += si[q][r];
                                si[q][r] = 0.0;
                            }
                        }
                        top[q] += si[q][NS - 1];
                        si[q][NS - 1] = 0.0;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < K; ++q) {
                const int k = (wave * K + q) * 64 + lane;
                if (k < icnt) {
                    double* dst = a.partial + (int64_t)ch * NS * n + ib + k;
#pragma unroll
                    for (int r = 0; r < NS - 1; ++r)
                        dst[(int64_t)r * n] = kTopLds ? s_top[kTopLds ? r : 0][kTopLds ? k : 0] : si[q][r];
                    dst[(int64_t)(NS - 1) * n] = -(kTop ? top[q] : si[q][NS - 1]);
                }
            }
        }
        if (!queue) break;   // one item per workgroup
        __syncthreads();
        if (tid == 0) s_item = (int)(gridDim.x + atomicAdd(queue, 1u));
        __syncthreads();
        item = s_item;
    }
}

// Ensembles: every cluster's items and their offsets (one workgroup).
__global__ void __launch_bounds__(kWG) pair_plan_kernel(SweepArgs a, PairShape sh, uint32_t* queue)
{
    const int tid = threadIdx.x, C = a.n_clusters;
    const int per = (C + kWG - 1) / kWG;
    const int c0 = tid * per < C ? tid * per : C;
    const int c1 = c0 + per < C ? c0 + per : C;
    int32_t local = 0, none = 0;
    int64_t inter = 0;
    for (int c = c0; c < c1; ++c) {
        const int64_t nc = a.offsets[c + 1] - a.offsets[c];
        const int nb = pair_blocks(nc, sh.bi);
        local += nb * pair_chunks(sh, pair_row(nb, 0, sh.k));
        inter += nc * nc;
    }
    int32_t total;
    int32_t base = block_exscan_sum_max(local, &total, &inter, &none);
    for (int c = c0; c < c1; ++c) {
        a.item_off[c] = base;
        const int nb = pair_blocks(a.offsets[c + 1] - a.offsets[c], sh.bi);
        base += nb * pair_chunks(sh, pair_row(nb, 0, sh.k));
    }
    if (tid == 0) {
        a.item_off[C] = total;
        a.plan->total_items = total;
        *queue = 0u;
        if (a.counters)
            atomicAdd((unsigned long long*)&a.counters[1], (unsigned long long)inter);
    }
}

// Adds every particle's partial sums: kGroups threads a particle, each the
// slots g, g + kGroups, ... two at a time (half the roundings at the sum's
// size), then the groups in pairs.
template <bool POT>
__global__ void __launch_bounds__(kWG) pair_reduce_kernel(SweepArgs a, PairShape sh)
{
    constexpr int NS = PairI<POT>::NS;
    constexpr int kGroups = 4, kPart = kWG / kGroups;
    __shared__ double s_s[kGroups - 1][NS][kPart];
    const int tid = threadIdx.x, g = tid / kPart, l = tid % kPart;
    const int64_t n = a.n;
    const int64_t p0 = (int64_t)blockIdx.x * kPart;
    const int64_t p = p0 + l;
    int64_t cb = 0, ce = n;
    if (a.n_clusters > 1) {
        int c = upper_bound_i64(a.offsets, a.n_clusters + 1, p0) - 1;
        while (p < n && p >= a.offsets[c + 1]) ++c;
        cb = a.offsets[c];
        ce = a.offsets[c + 1];
    }
    double s[NS];
#pragma unroll
    for (int r = 0; r < NS; ++r) s[r] = 0.0;
    if (p < n) {
        const int nb = pair_blocks(ce - cb, sh.bi);
        const int ab = (int)((p - cb) / sh.bi);
        const int ni = pair_chunks(sh, pair_row(nb, ab, sh.k));
        const int nj = (nb - 1) / 2 + ((nb & 1) == 0 && ab >= nb / 2 ? 1 : 0);
        const int cnt = ni + nj;
        for (int k = g; k < cnt; k += 2 * kGroups) {
            const int k2 = k + kGroups;
            const double* q0 = a.partial + (int64_t)(k < ni ? k : sh.nch + k - ni) * NS * n + p;
            const double* q1 = k2 < cnt
                ? a.partial + (int64_t)(k2 < ni ? k2 : sh.nch + k2 - ni) * NS * n + p : q0;
            double v0[NS], v1[NS];
#pragma unroll
            for (int r = 0; r < NS; ++r) {
                v0[r] = q0[(int64_t)r * n];
                v1[r] = q1[(int64_t)r * n];
            }
#pragma unroll
            for (int r = 0; r < NS; ++r) s[r] += v0[r] + (k2 < cnt ? v1[r] : 0.0);
        }
    }
    if (g > 0) {
#pragma unroll
        for (int r = 0; r < NS; ++r) s_s[g - 1][r][l] = s[r];
    }
    __syncthreads();
    if (a.n_clusters == 1 && a.counters && blockIdx.x == 0 && tid == 0)
        atomicAdd((unsigned long long*)&a.counters[1], (unsigned long long)(n * n));
    if (g > 0 || p >= n) return;
    static_assert(kGroups == 4, "added in pairs");
#pragma unroll
    for (int r = 0; r < NS; ++r) s[r] = (s[r] + s_s[0][r][l]) + (s_s[1][r][l] + s_s[2][r][l]);
    if constexpr (POT) {
        a.pot[p] = s[0];
    } else {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            a.acc[d * n + p] = s[d];
            if (a.jerk) a.jerk[d * n + p] = s[3 + d];
        }
        if (a.pot) a.pot[p] = s[6];
    }
}

// Chunk bounds of a row of u tiles, nb rows, on `slots` workgroups at a
// time: each level takes 1 / share of an even part of what is left, so that
// the items that start last are short.  (The two workgroups of a compute
// unit do not advance evenly: the older one is served first, and one left
// alone on its unit reaches about 0.7 of the pair rate.  N = 65536: 3.24 ms
// with these levels, 3.70 ms with 512 equal items for 512 places.)
void guided_levels(PairShape* sh, int u, int nb, int slots, double share, int longest)
{
    for (int qmin = 1;; ++qmin) {
        int c = 0, done = 0;
        while (done < u && c < kPairMaxLevels) {
            const int q = std::max(
                qmin, std::min(longest, (int)std::ceil((double)(u - done) * nb / (slots * share))));
            sh->lev[c++] = (int16_t)done;
            done += std::min(q, u - done);
        }
        sh->nch = c;
        sh->lev[c] = (int16_t)done;
        if (done >= u) return;
    }
}

}  // namespace

int64_t pair_partial_doubles(const PairShape& sh, int64_t n, int64_t n_cmax, bool pot_only)
{
    const int nb = pair_blocks(n_cmax, sh.bi);
    return (int64_t)(sh.nch + nb / 2) * (pot_only ? 1 : 7) * n;
}

bool pair_shape(int64_t n, int n_clusters, int64_t n_cmax, int n_cu, bool pot_only, PairShape* sh)
{
    std::memset(sh, 0, sizeof *sh);
    if (n_clusters > 1) {
        const double inter = (double)n * (double)n / n_clusters;   // at least this many
        if (n_cmax > kPairMaxCluster || n_clusters > kLdsClusters ||
            inter < (n_clusters < kPairMany ? kPairEnsemble : kPairManyEnsemble) ||
            n / n_clusters < kPairMeanCluster)
            return false;
        sh->k = 3;
        sh->w = 1;
        sh->bi = 64 * sh->k * sh->w;
        const int u = pair_row(pair_blocks(n_cmax, sh->bi), 0, sh->k);
        const int fill = (int)(inter / (2.0 * sh->bi * 64) / (16.0 * n_cu)) + 1;
        const int q = std::max(std::min(fill, kPairRun),
                               (u + kPairClusterSlots - 1) / kPairClusterSlots);
        int c = 0;
        for (int done = 0; done < u; done += q) sh->lev[c++] = (int16_t)done;
        sh->nch = c;
        sh->lev[c] = (int16_t)u;
        return true;
    }
    if (n < (pot_only ? kPairMinPot : kPairMin) || n > kPairMaxN) return false;
    sh->w = n >= (pot_only ? kPairWidePot : kPairWide) ? 4 : 1;
    sh->k = sh->w == 4 || n >= kPairFour ? 4 : 3;
    sh->bi = 64 * sh->k * sh->w;
    const int nb = pair_blocks(n, sh->bi);
    guided_levels(sh, pair_row(nb, 0, sh->k), nb, n_cu * (8 / sh->w),
                  sh->w == 4 || pot_only ? 1.5 : 1.0,
                  pair_two_levels(sh->k, pot_only) ? INT32_MAX : kPairRun);
    sh->items = nb * sh->nch;
    return true;
}

// The whole pair sweep.  queue: one device word (ensembles).
hipError_t launch_pairs(const SweepArgs& a, const PairShape& sh, uint32_t* queue, int n_cu,
                        bool pot_only, hipStream_t st, const hipEvent_t* marks)
{
    const bool many = a.n_clusters > 1;
    if (many) hipLaunchKernelGGL(pair_plan_kernel, dim3(1), dim3(kWG), 0, st, a, sh, queue);
    if (marks) {
        const hipError_t e = hipEventRecord(marks[0], st);
        if (e != hipSuccess) return e;
    }
    typedef void (*Fn)(SweepArgs, PairShape, uint32_t*);
    Fn f;
    if (sh.w == 4) f = pot_only ? pair_sweep_kernel<4, 4, true> : pair_sweep_kernel<4, 4, false>;
    else if (sh.k == 4) f = pot_only ? pair_sweep_kernel<4, 1, true> : pair_sweep_kernel<4, 1, false>;
    else f = pot_only ? pair_sweep_kernel<3, 1, true> : pair_sweep_kernel<3, 1, false>;
    const int grid = many ? n_cu * 8 : sh.items;
    hipLaunchKernelGGL(f, dim3(grid), dim3(64 * sh.w), 0, st, a, sh, many ? queue : nullptr);
    if (marks) {
        const hipError_t e = hipEventRecord(marks[1], st);
        if (e != hipSuccess) return e;
    }
    const int rgrid = (int)((a.n + kWG / 4 - 1) / (kWG / 4));
    if (pot_only)
        hipLaunchKernelGGL(pair_reduce_kernel<true>, dim3(rgrid), dim3(kWG), 0, st, a, sh);
    else
        hipLaunchKernelGGL(pair_reduce_kernel<false>, dim3(rgrid), dim3(kWG), 0, st, a, sh);
    return hipGetLastError();
}

}  // namespace hm
