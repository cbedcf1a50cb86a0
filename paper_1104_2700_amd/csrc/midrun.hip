// Block steps of one system of kSmallRunMax to kMidRunMax particles (FP64),
// many in one launch.
//
// Such a run's blocks are mostly tiny (N = 16384: half of them below 16
// particles), and a step is then the latency of three kernels: 17 us at
// N = 1600, 20.5 at 4096, 22.6 at 16384 against 0.1, 0.3 and 2 us of
// arithmetic.  Here P rows of Q workgroups, one a compute unit, stay for a
// whole batch of steps: 10.9, 10.9 and 14.7 us.  Workgroup (p, q) holds slice
// q of the particles (registers; what the sweep reads, predicted, in LDS), so
// every row holds the whole system; row p sweeps the active positions p,
// p + P, ..., each of its workgroups over its slice, and every workgroup
// corrects the active particles of its own slice (the P copies of a slice do
// the same).  Two exchanges a step, 2 to 3 us each: the slices' earliest
// times with their due particles, and the partial sums.  In larger blocks P
// copies of a slice reading the same partial sums are too much traffic: there
// each copy corrects its share, and the corrected particles are a third
// exchange.
//
// The exchange.  Words of eight bytes, each half payload and half the step's
// tag, by relaxed device-scope stores and loads: a reader polls the words it
// needs until they bear the tag, so that no flag, no order among stores and
// no wait for them is needed (a flag behind its data costs a further trip to
// memory on either side).  Every workgroup waits for every header of a step,
// and sends its own when it has read the last step's partial sums: headers
// and due particles alternate between two buffers (a slow reader may still be
// at the last step's when the next one's arrive), the others need one.
//
// No wait is without end, and a launch that is given up leaves the state as
// it was: see smallrun.hip.  So does a block whose plan has chunks that do not
// tile a slice or have no room (none has with the default tuning's rules).
//
// The sums are the ones of the step-by-step path bit for bit: the plan's
// lanes and chunks, its reduction's order, and the same corrector.
#include "correct.h"
#include "hermite_internal.h"
#include "pair.h"
#include "plan.h"
#include "run_common.h"

namespace hm {
namespace {

constexpr int kWaves = kMidThreads / 64;
// Active particles of a row staged at a time: 64 where their sums over a
// slice's chunks wait in LDS, a particle a thread where they go straight out.
// (There plans have few lanes and long chunks, and a wave takes 64 / lanes
// particles and a chunk: from 64 particles one wave of the eight had work.
// N = 16384: 8192 active 534 us a step, now 209; 4096 146, now 112.)
constexpr int kStage = 64, kStageMax = kMidThreads;
constexpr int kBatch = 64;       // active particles of a slice corrected at a time
// From so many lines read by all copies on, the copies share the work: a
// third exchange costs 1.5 to 3 us, and 65536 lines are 8 MB through the
// memory side (flat from 32768 to 131072: 15.0 to 15.3 us a step at N =
// 16384, 12.9 to 12.6 at 4096).
constexpr int64_t kShareLines = 65536;
constexpr int kRecWords = 29;    // a corrected particle: 14 values and the clamped flag
static_assert(kMidThreads >= 8 * kBatch && kMidThreads >= 8 * kStage, "lanes of a batch");
static_assert(kMidMaxSlices <= 16, "16 lanes for the slices' sums");

struct Spin {            // a bounded wait
    int64_t patience;
    const int64_t* verdict;
    int64_t launch;
    int64_t t0 = 0;
    int k = 0;
    __device__ bool over()
    {
        if (++k < 256) return false;
        const int64_t now = wall_clock64();
        if (t0 == 0) t0 = now;
        return now - t0 > patience || given_up(verdict, launch);
    }
};

__device__ __forceinline__ void put(uint64_t* p, uint32_t payload, uint32_t tag)
{
    __hip_atomic_store(p, (uint64_t)payload | ((uint64_t)tag << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t get(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void put_double(uint64_t* p, double v, uint32_t tag)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    put(p, (uint32_t)b, tag);
    put(p + 1, (uint32_t)(b >> 32), tag);
}

__device__ __forceinline__ double two_words(uint64_t lo, uint64_t hi)
{
    return __longlong_as_double((long long)((hi << 32) | (lo & 0xffffffffull)));
}

// K words at p with the tag; false when the wait is over.
template <int K>
__device__ __forceinline__ bool take(const uint64_t* p, uint32_t tag, Spin& spin, uint64_t (&w)[K])
{
    for (;;) {
        bool ok = true;
#pragma unroll
        for (int k = 0; k < K; ++k) w[k] = get(p + k);
#pragma unroll
        for (int k = 0; k < K; ++k) ok = ok && (uint32_t)(w[k] >> 32) == tag;
        if (ok) return true;
        if (spin.over()) return false;
        __builtin_amdgcn_s_sleep(1);
    }
}

template <int O>
__device__ __forceinline__ void sum_step(double (&o)[7])
{
#pragma unroll
    for (int u = 0; u < 7; ++u) o[u] = lane_sum<O>(o[u]);
}

// The plan of every block size: log2 (lanes) | 8 log2 (tiles of a chunk), or
// kNoPlan where the chunks do not tile a slice or have no room.  A wave a
// size (a thread a size: 70 us at N = 16384, its divisions one after another).
constexpr int kNoPlan = 255;
__global__ void __launch_bounds__(kWG) mid_plan_kernel(MidRunArgs e, SweepArgs sa)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int na = (int)blockIdx.x * (kWG / 64) + wave + 1;
    if (na > (int)sa.n) return;
    int32_t L, ti;
    int64_t jc;
    plan_split_wave(sa, na, 1, &L, &ti, &jc);
    if (e.model && split_by_model(sa, na)) split_for_sizes_wave(sa, na, &L, &ti, &jc);
    const bool ok = jc <= kMidSlice && kMidSlice % jc == 0 &&
                    (int64_t)((na + e.rows - 1) / e.rows) * (kMidSlice / jc) <= e.partial_lines;
    if ((threadIdx.x & 63) != 0) return;
    e.plans[na] = ok ? (uint8_t)((31 - __clz(L)) | (31 - __clz((int)(jc / kTJ))) << 3)
                     : (uint8_t)kNoPlan;
}

__global__ void __launch_bounds__(kMidThreads) mid_run_kernel(SmallRunArgs r, MidRunArgs e)
{
    constexpr int KP = kMidSlice / kMidThreads;    // particles of a thread
    constexpr int S = kMidSlice;
    __shared__ double s_p[7][S];                   // x, v at the block time; m
    __shared__ double s_i[6][kStageMax];
    __shared__ int32_t s_ii[kStageMax];
    __shared__ double s_c[kStage * (S / kTJ)][7];   // their sums over each chunk
    __shared__ double s_old[kBatch][7];            // dt, a, j
    __shared__ int32_t s_oi[kBatch];
    __shared__ double s_f[kBatch][8];
    __shared__ double s_new[kBatch][13];
    __shared__ int64_t s_min[kWaves];
    __shared__ int32_t s_cnt[kWaves];
    __shared__ int64_t s_hmin[kMidMaxSlices];
    __shared__ int32_t s_hcnt[kMidMaxSlices];
    __shared__ int32_t s_stop;
    __shared__ int32_t s_hist[33];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grid = (int)gridDim.x, Q = e.slices, P = e.rows;
    // consecutive workgroups go to the eight XCDs in turn: a row is kept on
    // one, and so are the headers of a line
    auto place = [&](int b) { return grid % 8 == 0 ? (b % 8) * (grid / 8) + b / 8 : b; };
    const int stride = mid_header_words(grid) / 8, words = 8 * stride;
    const int g = place((int)blockIdx.x);
    const int my_word = (int)(blockIdx.x % 8) * stride + (int)(blockIdx.x / 8);
    const int its_word = (tid % 8) * stride + tid / 8;   // workgroup tid's
    const int p = g / Q, q = g - p * Q;
    const int n = (int)r.n;
    const double tick = ldexp(1.0, -r.tick_bits);

    // this thread's particles: j = S q + kMidThreads k + tid; past the end
    // massless ones far away, never due
    double x[KP][3], v[KP][3], a[KP][3], jk[KP][3];
    int64_t t[KP], dt[KP];
#pragma unroll
    for (int k = 0; k < KP; ++k) {
        const int j = S * q + kMidThreads * k + tid;
        const bool ok = j < n;
        const int jj = ok ? j : 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            x[k][d] = ok ? r.x[d * (int64_t)n + jj] : 1.0e30;
            v[k][d] = ok ? r.v[d * (int64_t)n + jj] : 0.0;
            a[k][d] = ok ? r.a[d * (int64_t)n + jj] : 0.0;
            jk[k][d] = ok ? r.j[d * (int64_t)n + jj] : 0.0;
        }
        s_p[6][kMidThreads * k + tid] = ok ? r.m[jj] : 0.0;
        t[k] = ok ? r.t[jj] : 0;
        dt[k] = ok ? r.dt[jj] : 0;
    }
    if (tid < 33) s_hist[tid] = 0;
    if (tid == 0) s_stop = r.patience < 0 ? 1 : 0;
    __syncthreads();
    int64_t T = 0, inter = 0, done_steps = 0, last_T = 0;
    int32_t na = 0, last_na = 0, clamped = 0, bad = 0;
    bool gave_up = s_stop != 0;
    int32_t to_check = r.check_every;
    // z / P, z < 65536
    auto by_rows = [&](int z) { return (int)__umulhi((uint32_t)z, e.rows_inverse); };
    auto chunks = [&](int plan) {
        const int lg = 8 + ((plan >> 3) & 3);   // log2 of a chunk (any value for kNoPlan)
        return (n + (1 << lg) - 1) >> lg;
    };

    for (int64_t step = 1; step <= r.steps && !gave_up; ++step) {
        const uint32_t tag = (uint32_t)(r.epoch + step);
        const int par = (int)(step & 1);
        // ---- this slice's earliest time and its due particles ----------------
        int32_t wrong = 0;
        if (to_check-- == 0) {   // before step check_every + 1, 2 check_every + 1, ...
            to_check = r.check_every - 1;
            wrong = __syncthreads_or(non_finite(x, v, a, jk) ? 1 : 0) ? 1 : 0;
        }
        int64_t en[KP], mn = INT64_MAX;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            const bool ok = S * q + kMidThreads * k + tid < n;
            en[k] = ok ? t[k] + dt[k] : INT64_MAX;
            mn = min_i64(mn, en[k]);
        }
        mn = wave_min_i64(mn);
        unsigned long long due[KP];
        int32_t c = 0;
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            due[k] = __ballot(en[k] == mn && mn != INT64_MAX);
            c += __popcll(due[k]);
        }
        if (lane == 0) {
            s_min[wave] = mn;
            s_cnt[wave] = c;
        }
        __syncthreads();
        int64_t mine_T = s_min[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) mine_T = min_i64(mine_T, s_min[w]);
        int32_t base = 0, mine_cnt = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int32_t cw = s_min[w] == mine_T ? s_cnt[w] : 0;
            base += w < wave ? cw : 0;
            mine_cnt += cw;
        }
        uint64_t* hdr = e.header + par * 3 * words;
        if (tid == 0) {
            put(hdr + my_word, (uint32_t)mine_cnt | ((uint32_t)wrong << 31), tag);
            put(hdr + words + my_word, (uint32_t)mine_T, tag);
            put(hdr + 2 * words + my_word, (uint32_t)((uint64_t)mine_T >> 32), tag);
        }
        bool act[KP];
        int32_t slot[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            act[k] = mn == mine_T && ((due[k] >> lane) & 1ull) != 0;
            slot[k] = base + __popcll(due[k] & ((1ull << lane) - 1ull));
            base += mn == mine_T ? __popcll(due[k]) : 0;
            // the first slots to this row, the others once for all rows
            if (act[k] && (slot[k] < kMidRowSlots || slot[k] - by_rows(slot[k]) * P == p)) {
                OldState o;
                o.i = S * q + kMidThreads * k + tid;
                o.t = t[k];
                o.dt = dt[k];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    o.x[d] = x[k][d];
                    o.v[d] = v[k][d];
                    o.a[d] = a[k][d];
                    o.j[d] = jk[k][d];
                }
                double xp[3], vp[3];
                predict_old(o, mine_T, tick, xp, vp);
                uint64_t* w = slot[k] < kMidRowSlots
                    ? e.row_due + (((int64_t)par * grid + g) * kMidRowSlots + slot[k]) * kMidLine
                    : e.all_due + ((int64_t)par * Q * S + S * q + slot[k]) * kMidLine;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    put_double(w + 2 * d, xp[d], tag);
                    put_double(w + 6 + 2 * d, vp[d], tag);
                }
                put(w + 12, (uint32_t)o.i, tag);
            }
        }
        // ---- every workgroup's header ------------------------------------------
        if (tid < grid) {
            Spin spin{step == 1 ? r.arrival : r.patience, e.verdict, r.launch};
            uint64_t w[1], lo[1], hi[1];
            bool ok = take(hdr + its_word, tag, spin, w);
            const int qq = place(tid) - p * Q;
            if (qq >= 0 && qq < Q) {
                ok = take(hdr + words + its_word, tag, spin, lo) && ok;
                ok = take(hdr + 2 * words + its_word, tag, spin, hi) && ok;
                s_hmin[qq] = (int64_t)((hi[0] << 32) | (lo[0] & 0xffffffffull));
                s_hcnt[qq] = (int32_t)(uint32_t)w[0];
            }
            if (!ok) s_stop = 1;
        }
        __syncthreads();
        if (s_stop) {
            gave_up = true;
            break;
        }
        // the block: T, and the slices' positions in it (a lane a slice)
        const int64_t hm = lane < Q ? s_hmin[lane] : INT64_MAX;
        const int32_t hc = lane < Q ? s_hcnt[lane] : 0;
        if (__any(hc < 0)) {
            bad = 1;
            break;
        }
        T = wave_min_i64(hm);
        if (T > r.T_end) {
            na = 0;
            break;
        }
        const int32_t in = hm == T ? hc : 0;
        const int32_t upto = wave_inscan(in);
        na = __builtin_amdgcn_readlane(upto, 63);
        const int32_t first = upto - in;             // lane: the slice's first position
        const int32_t my_first = __builtin_amdgcn_readlane(first, q);
        const int32_t my_na = __builtin_amdgcn_readlane(in, q);
        // ---- the plan, the row's particles, the prediction ----------------------
        const int plan = e.plans[na];
        const int mine = na > p ? by_rows(na - 1 - p) + 1 : 0;   // positions p, p + P, ...
        const int ch = chunks(plan);                        // of the system
        const bool by_thread = thread_reduce(ch, na);
        const int batch = by_thread ? kStageMax : kStage;
        auto stage = [&](int r0) {
            const int rr = r0 + tid, pos = p + P * rr;
            if (64 * wave >= batch || r0 + 64 * wave >= mine) return;
            int sl = 0, f = 0;
            for (int k = 0; k < Q; ++k) {
                const int fk = __builtin_amdgcn_readlane(first, k);
                const int ck = __builtin_amdgcn_readlane(in, k);
                sl = pos >= fk && pos < fk + ck ? k : sl;
                f = pos >= fk && pos < fk + ck ? fk : f;
            }
            if (rr < mine) {
                const int s = pos - f;
                const uint64_t* w = s < kMidRowSlots
                    ? e.row_due + (((int64_t)par * grid + p * Q + sl) * kMidRowSlots + s) * kMidLine
                    : e.all_due + ((int64_t)par * Q * S + S * sl + s) * kMidLine;
                Spin spin{r.patience, e.verdict, r.launch};
                uint64_t u[13];
                if (!take(w, tag, spin, u)) s_stop = 1;
#pragma unroll
                for (int d = 0; d < 6; ++d) s_i[d][tid] = two_words(u[2 * d], u[2 * d + 1]);
                s_ii[tid] = (int32_t)(uint32_t)u[12];
            }
        };
        stage(0);
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            OldState o;
            o.i = 0;
            o.t = t[k];
            o.dt = dt[k];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                o.x[d] = x[k][d];
                o.v[d] = v[k][d];
                o.a[d] = a[k][d];
                o.j[d] = jk[k][d];
            }
            double xp[3], vp[3];
            predict_old(o, T, tick, xp, vp);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                s_p[d][kMidThreads * k + tid] = xp[d];
                s_p[3 + d][kMidThreads * k + tid] = vp[d];
            }
        }
        __syncthreads();
        if (s_stop) {
            gave_up = true;
            break;
        }
        if (plan == kNoPlan) {   // in every workgroup
            gave_up = true;
            break;
        }
        const int lg = plan & 7, L = 1 << lg;
        const int jc = kTJ << (plan >> 3);
        constexpr int lS = 2;
        static_assert(kTJ == 256 && S == kTJ << lS, "a slice in tiles");
        const int lper = lS - (plan >> 3), per = 1 << lper;   // chunks of a slice
        const int nch = min(per, ch - q * per);
        // ---- the sweep: a wave 64 / L of the row's particles and a chunk -------
        // (where the reduction is a butterfly over the chunks, a slice's chunks
        // are its first steps, taken here: a slice's sums then are one line)
        const int sub = lane & (L - 1);
        const int G = 64 >> lg;
        for (int r0 = 0; r0 < mine; r0 += batch) {
            if (r0 > 0) {
                __syncthreads();
                stage(r0);
                __syncthreads();
                if (s_stop) break;
            }
            const int cnt = min(batch, mine - r0);
            const int items = ((cnt + G - 1) >> (6 - lg)) << lper;
            for (int it = wave; it < items; it += kWaves) {
                const int grp = it >> lper, cc = it & (per - 1);
                if (cc >= nch) continue;
                const int rr = grp * G + (lane >> lg);
                const bool ok = rr < cnt;
                const int ri = ok ? rr : 0;
                const I64 I{s_i[0][ri], s_i[1][ri], s_i[2][ri], s_i[3][ri], s_i[4][ri], s_i[5][ri]};
                const int self = s_ii[ri] - S * q;
                SumD A;
                A.zero();
                const int j0 = cc * jc + sub;
                for (int k0 = 0; k0 < jc; k0 += kTJ) {   // a tile's sum, then the tiles'
                    SumD B;
                    B.zero();
                    for (int k = k0; k < k0 + kTJ; k += 4 * L) {
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int j = j0 + k + u * L;
                            pair_f64<true>(I, r.eps2, s_p[0][j], s_p[1][j], s_p[2][j], s_p[3][j],
                                           s_p[4][j], s_p[5][j], s_p[6][j], j == self, B);
                        }
                    }
                    A.add(B);
                }
                double* c = s_c[by_thread ? 0 : rr * per + cc];
                uint64_t* w = e.partial +
                    ((int64_t)g * e.partial_lines + ((r0 + rr) << lper) + cc) * kMidLine;
                if (L >= 8) {
                    const double o[8] = {A.ax, A.ay, A.az, A.jx, A.jy, A.jz, -A.pp, 0.0};
                    const double f = lanes_sum8(o, L);
                    const int u = summed8_index();
                    if (ok && sub < 8 && u < 7) {
                        if (by_thread) put_double(w + 2 * u, f, tag);
                        else c[u] = f;
                    }
                } else {
                    double o[7] = {A.ax, A.ay, A.az, A.jx, A.jy, A.jz, -A.pp};
                    if (L > 1) sum_step<1>(o);
                    if (L > 2) sum_step<2>(o);
                    if (ok && sub == 0) {
#pragma unroll
                        for (int u = 0; u < 7; ++u) {
                            if (by_thread) put_double(w + 2 * u, o[u], tag);
                            else c[u] = o[u];
                        }
                    }
                }
            }
            if (by_thread) continue;
            __syncthreads();
            const int rr = tid >> 3, u = tid & 7;
            if (rr < cnt && u < 7) {
                const double* c = &s_c[rr * per][u];
                auto chunk = [&](int k) { return k < nch ? 0.0 + c[k * 7] : 0.0; };
                double f = chunk(0);
                if (per > 1) f += chunk(1);
                if (per > 2) f += chunk(2) + chunk(3);
                put_double(e.partial + ((int64_t)g * e.partial_lines + r0 + rr) * kMidLine + 2 * u,
                           f, tag);
            }
        }
        // every wave's partial sums are on their way before any wave polls: a
        // compute unit full of polling waves may not let another one's store
        // pass (oldest first), and they would wait for each other
        __builtin_amdgcn_s_barrier();
        // ---- the sums of this slice's active particles, and the corrector --------
        // small blocks: every copy of a slice for itself; otherwise its copies
        // in turn, with a third exchange (see the top)
        const int lines = by_thread ? ch : Q;        // of a particle
        const bool share = (int64_t)na * lines * P > kShareLines;
        const int step_s = share ? P : 1, first_s = share ? p : 0;
        const int list = share ? (my_na > p ? by_rows(my_na - 1 - p) + 1 : 0) : my_na;
        const int q_first = by_rows(my_first), q_rest = my_first - q_first * P;
        // the partial sums of the slice's slot s over slice 0
        const int64_t next = e.partial_lines * kMidLine;   // from there to the next slice
        auto partial_of = [&](int s) -> const uint64_t* {
            const int z = q_rest + s, zq = by_rows(z), rr = q_first + zq, row = z - zq * P;
            return e.partial + row * Q * next + (by_thread ? rr << lper : rr) * kMidLine;
        };
        for (int b0 = 0; b0 < list; b0 += kBatch) {
            const int cnt = min(kBatch, list - b0);
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                const int zs = share ? by_rows(slot[k]) : slot[k];
                const int s = zs - b0;
                if (act[k] && slot[k] - zs * step_s == first_s && s >= 0 && s < cnt) {
                    s_oi[s] = kMidThreads * k + tid;
                    s_old[s][0] = __longlong_as_double(dt[k]);
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        s_old[s][1 + d] = a[k][d];
                        s_old[s][4 + d] = jk[k][d];
                    }
                }
            }
            Spin spin{r.patience, e.verdict, r.launch};
            if (by_thread) {
                const int s = tid >> 3, u = tid & 7;
                if (s < cnt && u < 7) {
                    const uint64_t* w = partial_of(first_s + step_s * (b0 + s)) + 2 * u;
                    double f = 0.0;
                    for (int k = 0; k < ch; k += kReduceBatch) {
                        uint64_t lo[kReduceBatch], hi[kReduceBatch];
                        for (;;) {
                            bool ok = true;
#pragma unroll
                            for (int z = 0; z < kReduceBatch; ++z) {
                                const int kk = k + z < ch ? k + z : ch - 1;
                                const uint64_t* wk =
                                    w + (kk >> lper) * next + (kk & (per - 1)) * kMidLine;
                                lo[z] = get(wk);
                                hi[z] = get(wk + 1);
                            }
#pragma unroll
                            for (int z = 0; z < kReduceBatch; ++z)
                                ok = ok && (uint32_t)(lo[z] >> 32) == tag &&
                                     (uint32_t)(hi[z] >> 32) == tag;
                            if (ok) break;
                            if (spin.over()) {
                                s_stop = 1;
                                break;
                            }
                            __builtin_amdgcn_s_sleep(1);
                        }
#pragma unroll
                        for (int z = 0; z < kReduceBatch; ++z)
                            f += k + z < ch ? two_words(lo[z], hi[z]) : 0.0;
                    }
                    s_f[s][u] = f;
                }
            } else {
                for (int s0 = 4 * wave; s0 < cnt; s0 += 4 * kWaves) {   // 16 lanes each
                    const int s = s0 + (lane >> 4), k = lane & 15;
                    double o[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
                    if (s < cnt && k < Q) {
                        uint64_t w[14];
                        if (!take(partial_of(first_s + step_s * (b0 + s)) + k * next, tag, spin, w))
                            s_stop = 1;
#pragma unroll
                        for (int u = 0; u < 7; ++u) o[u] = two_words(w[2 * u], w[2 * u + 1]);
                    }
                    const double f = lanes_sum8(o, 16);
                    if (s < cnt && k < 8) s_f[s][summed8_index()] = f;
                }
            }
            __syncthreads();
            if (s_stop) break;
            // a quad of lanes a particle, a lane a component (the fourth: the
            // potential), then a norm each
            if (tid < 4 * kBatch && 4 * cnt > (tid & ~63)) {
                const bool ok = (tid >> 2) < cnt;
                const int s = ok ? tid >> 2 : 0, d = lane & 3, dd = d < 3 ? d : 0;
                const int64_t dt_old = __double_as_longlong(s_old[s][0]);
                const double f0 = s_f[s][d < 3 ? d : 6], f1 = s_f[s][3 + dd];
                const StepPowers sp = step_powers(dt_old, tick);
                double x1, v1, s1, c1;
                correct_component(sp, s_old[s][1 + dd], s_old[s][4 + dd], f0, f1,
                                  s_p[dd][s_oi[s]], s_p[3 + dd][s_oi[s]], &x1, &v1, &s1, &c1);
                double u[3];
#pragma unroll
                for (int z = 0; z < 3; ++z) {
                    const double ua = quad_value(f0, z), uj = quad_value(f1, z);
                    const double us = quad_value(s1, z), uc = quad_value(c1, z);
                    u[z] = d == 0 ? ua : d == 1 ? uj : d == 2 ? us : uc;
                }
                const double nm = norm3(u[0], u[1], u[2]);
                const double crit = step_criterion(quad_value(nm, 0), quad_value(nm, 1),
                                                   quad_value(nm, 2), quad_value(nm, 3), r.eta,
                                                   r.form);
                int cl;
                const int64_t dn = quantize_dt(crit, r.tick_bits - log2_step(dt_old), T,
                                               r.tick_bits, r.k_min, r.k_max, &cl);
                if (ok && share) {
                    uint64_t* w = e.corrected +
                        ((int64_t)S * q + first_s + step_s * (b0 + s)) * 2 * kMidLine;
                    if (d < 3) {
                        put_double(w + 2 * d, x1, tag);
                        put_double(w + 6 + 2 * d, v1, tag);
                        put_double(w + 12 + 2 * d, f0, tag);
                        put_double(w + 18 + 2 * d, f1, tag);
                    } else {
                        put_double(w + 24, __longlong_as_double((long long)dn), tag);
                        put_double(w + 26, f0, tag);
                        put(w + 28, (uint32_t)cl, tag);
                    }
                } else if (ok) {
                    if (d < 3) {
                        s_new[s][d] = x1;
                        s_new[s][3 + d] = v1;
                        s_new[s][6 + d] = f0;
                        s_new[s][9 + d] = f1;
                    } else {
                        s_new[s][12] = __longlong_as_double((long long)dn);
                        if (p == 0) {
                            r.pot[S * q + s_oi[s]] = f0;
                            clamped += cl;
                        }
                    }
                }
            }
            if (b0 + kBatch < list || !share) __syncthreads();
            if (share) continue;
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                const int s = slot[k] - b0;
                if (act[k] && s >= 0 && s < cnt) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        x[k][d] = s_new[s][d];
                        v[k][d] = s_new[s][3 + d];
                        a[k][d] = s_new[s][6 + d];
                        jk[k][d] = s_new[s][9 + d];
                    }
                    dt[k] = __double_as_longlong(s_new[s][12]);
                    t[k] = T;
                }
            }
            if (b0 + kBatch < list) __syncthreads();
        }
        if (share) {
            // the corrected particles, by way of LDS (the predictions' place):
            // consecutive threads take consecutive words
            constexpr int kRec = 31, kRecs = (int)sizeof(double) * 6 * S / (4 * kRec);
            uint32_t* s_rec = (uint32_t*)&s_p[0][0];
            for (int b0 = 0; b0 < my_na; b0 += kRecs) {
                const int cnt = min(kRecs, my_na - b0);
                __syncthreads();
                const uint64_t* w = e.corrected + ((int64_t)S * q + b0) * 2 * kMidLine;
                Spin spin{r.patience, e.verdict, r.launch};
                for (int i = tid; i < cnt * 2 * kMidLine; i += 4 * kMidThreads) {
                    uint64_t u[4];
                    for (;;) {
                        bool ok = true;
#pragma unroll
                        for (int z = 0; z < 4; ++z) {
                            const int iz = i + z * kMidThreads;
                            const bool in_use = iz < cnt * 2 * kMidLine &&
                                                (iz & (2 * kMidLine - 1)) < kRecWords;
                            u[z] = get(w + (in_use ? iz : 0));
                        }
#pragma unroll
                        for (int z = 0; z < 4; ++z) ok = ok && (uint32_t)(u[z] >> 32) == tag;
                        if (ok) break;
                        if (spin.over()) {
                            s_stop = 1;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(1);
                    }
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        const int iz = i + z * kMidThreads, wz = iz & (2 * kMidLine - 1);
                        if (iz < cnt * 2 * kMidLine && wz < kRecWords)
                            s_rec[iz / (2 * kMidLine) * kRec + wz] = (uint32_t)u[z];
                    }
                }
                __syncthreads();
                if (s_stop) break;
#pragma unroll
                for (int k = 0; k < KP; ++k) {
                    const int s = slot[k] - b0;
                    if (!act[k] || s < 0 || s >= cnt) continue;
                    const uint32_t* u = s_rec + s * kRec;
                    auto value = [&](int z) { return two_words(u[2 * z], u[2 * z + 1]); };
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        x[k][d] = value(d);
                        v[k][d] = value(3 + d);
                        a[k][d] = value(6 + d);
                        jk[k][d] = value(9 + d);
                    }
                    dt[k] = __double_as_longlong(value(12));
                    t[k] = T;
                    if (p == 0) {
                        r.pot[S * q + kMidThreads * k + tid] = value(13);
                        clamped += (int32_t)u[28];
                    }
                }
            }
        }
        if (s_stop) {
            gave_up = true;
            break;
        }
        inter += (int64_t)na * n;
        ++done_steps;
        last_T = T;
        last_na = na;
        if (g == 0 && tid == 0) s_hist[32 - __clz(na)] += 1;
    }

    // ---- does the launch count? -------------------------------------------------
    __syncthreads();
    if (!gave_up) {
        const uint32_t tag = (uint32_t)(r.epoch + r.steps + 1);
        uint64_t* hdr = e.header + 2 * 3 * words;
        const int wrong = __syncthreads_or(non_finite(x, v, a, jk) ? 1 : 0) ? 1 : 0;
        if (tid == 0) put(hdr + my_word, (uint32_t)wrong, tag);
        uint64_t w[1] = {0};
        if (tid < grid) {
            Spin spin{r.patience, e.verdict, r.launch};
            if (!take(hdr + its_word, tag, spin, w)) s_stop = 1;
        }
        bad |= __syncthreads_or((int)((uint32_t)w[0] & 1u)) ? 1 : 0;
        gave_up = s_stop != 0;
    }
    __syncthreads();
    if (tid == 0) s_stop = settle(e.verdict, r.launch, !gave_up) ? 0 : 1;
    __syncthreads();
    const bool commit = s_stop == 0;
    if (commit && p == 0) {
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            const int j = S * q + kMidThreads * k + tid;
            if (j < n && done_steps > 0) {
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    r.x[d * (int64_t)n + j] = x[k][d];
                    r.v[d * (int64_t)n + j] = v[k][d];
                    r.a[d * (int64_t)n + j] = a[k][d];
                    r.j[d * (int64_t)n + j] = jk[k][d];
                }
                r.t[j] = t[k];
                r.dt[j] = dt[k];
            }
        }
        const int32_t cl = wave_sum_i32(clamped);
        if (lane == 0 && cl > 0)
            atomicAdd((unsigned long long*)&r.counters[2], (unsigned long long)cl);
    }
    if (g != 0) return;
    if (commit && tid < 33 && s_hist[tid] > 0)
        atomicAdd((unsigned long long*)&r.counters[kHistBase + tid],
                  (unsigned long long)s_hist[tid]);
    if (tid == 0) {
        if (commit && done_steps > 0) {
            atomicAdd((unsigned long long*)&r.counters[0], (unsigned long long)done_steps);
            atomicAdd((unsigned long long*)&r.counters[1], (unsigned long long)inter);
            r.counters[3] = last_T;
            r.counters[4] = last_na;
        }
        if (commit) {
            *r.na_out = na;
            *r.T_out = T;
        }
        SmallRunStatus* h = r.status;
        h->done = commit ? 1 : 0;
        h->steps = done_steps;
        h->interactions = inter;
        h->T = T;
        h->na = na;
        h->bad = bad;
        h->left = 0;
        h->launch = r.launch;
    }
}

}  // namespace

MidRunShape mid_run_shape(int64_t n, int n_cu)
{
    MidRunShape m;
    m.slices = (int)((n + kMidSlice - 1) / kMidSlice);
    m.rows = m.slices <= kMidMaxSlices ? std::min(n_cu, kMidThreads) / m.slices : 0;
    // of a workgroup: with at most 16 partial sums a particle (split_cost, or
    // up to 4096 particles of a tile or two a chunk) na <= 16 jc, and
    // (na / P + 1) (S / jc) <= 16 S / P + 8
    m.partial_lines = m.rows > 0 ? 16 * kMidSlice / m.rows + 16 : 0;
    return m;
}

hipError_t launch_mid_run(const SmallRunArgs& r, const MidRunArgs& e, const SweepArgs& sa,
                          hipStream_t st)
{
    const dim3 grid(e.rows * e.slices), wg(kMidThreads);
    hipLaunchKernelGGL(mid_plan_kernel, dim3((unsigned)((r.n + kWG / 64 - 1) / (kWG / 64))),
                       dim3(kWG), 0, st, e, sa);
    hipLaunchKernelGGL(mid_run_kernel, grid, wg, 0, st, r, e);
    return hipGetLastError();
}

}  // namespace hm
