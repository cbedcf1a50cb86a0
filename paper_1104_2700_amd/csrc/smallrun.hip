// Block steps of one small system (up to kSmallRunMax particles, FP64), many
// in one launch.
//
// A block step of a small system is latency: at N = 1024 two kernels of 10
// and 4.5 us and the gaps between them move 16 us for 5e4 interactions.  Here
// kSmallRunGrid workgroups stay on the chip for a whole batch of steps.
// Every one of them holds the whole state in registers (a wave a chunk of 256
// particles, four a lane) and does the same selection, so nothing but the
// corrected particles has to travel: a workgroup sweeps and corrects the
// active positions p = g, g + grid, ..., publishes them, and takes everyone's.
//
// The exchange.  Records and flags are relaxed device-scope atomics (they go
// past the per-XCD L2s): a workgroup writes its records and, behind a release
// fence, sets its flag to the step's number; it goes on when all flags have
// it, behind an acquire fence.  (The fences' cache operations move nothing
// here, but only they order the accesses in the memory model: 5.73 us a step
// at N = 1024 with a bare wait for the writes, 5.82 with the release, 6.15
// with both.)  Records alternate between two buffers: nobody can write step
// s + 2 before all flags have s + 1, which a workgroup sets after it has
// read step s.  A round of this among 64 workgroups with 64 records takes
// 2.3 us without the fences (measured alone; 16 workgroups 2.25, 8 on one XCD
// 1.7).
//
// No wait is without end: a workgroup that waits longer than `arrival` in the
// first step, or `patience` later, gives up, and the launch with it.  Whether the launch counts is settled by
// one word that the first to know sets (all steps done by all, or given up);
// only then is anything of the state but the potentials written, so a launch
// that was given up leaves the state as it was and the host takes the steps
// one by one (which write the same potentials again).
//
// The sums are the ones of the step-by-step path bit for bit: 64 lanes a
// particle, lane l adding j = l, l + 64, ... of a 256-particle tile, the
// lanes' butterfly, then the tiles in order, and the same corrector.
#include "correct.h"
#include "hermite_internal.h"
#include "pair.h"
#include "plan.h"
#include "run_common.h"

namespace hm {
namespace {

constexpr int kPer = kTJ / 64;                     // particles of a lane
static_assert(kSmallRunMax == 6 * kTJ, "at most six waves");
constexpr int kMaxSlots = kSmallRunMax / kSmallRunGrid;

// One wave: waits until every workgroup's flag is at least `want`.  False
// when that takes longer than `patience` (at once when that is negative) or
// another workgroup has given up.
__device__ bool wait_all(const int64_t* flags, int64_t want, int64_t patience, int64_t launch)
{
    const int lane = threadIdx.x & 63;
    static_assert(kSmallRunGrid == 64, "one flag a lane");
    const int64_t* f = flags + lane * kSmallRunLine;
    if (patience < 0) return false;
    for (int k = 0; k < 64; ++k)
        if (__all(get(f) >= want)) return true;
    const int64_t t0 = wall_clock64();
    while (!__all(get(f) >= want))
        if (wall_clock64() - t0 > patience ||
            __any(given_up(flags + kSmallRunGrid * kSmallRunLine, launch)))
            return false;
    return true;
}

struct Rec {             // an active particle of this workgroup, from its owner
    OldState o;
    double xp[3], vp[3];
    int pos;
};

// This wave's tile's part of the sums of one active particle.
__device__ __forceinline__ void sweep_slot(const Rec& q, const double (&px)[kPer][3],
                                           const double (&pv)[kPer][3], const double (&m)[kPer],
                                           int wave, double eps2, double* part)
{
    const int lane = threadIdx.x & 63;
    const I64 I{q.xp[0], q.xp[1], q.xp[2], q.vp[0], q.vp[1], q.vp[2]};
    const int i = q.o.i;
    SumD S;
    S.zero();
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        pair_f64<true>(I, eps2, px[k][0], px[k][1], px[k][2], pv[k][0], pv[k][1], pv[k][2], m[k],
                       kTJ * wave + 64 * k + lane == i, S);
    const double o[8] = {S.ax, S.ay, S.az, S.jx, S.jy, S.jz, -S.pp, 0.0};
    const double f = lanes_sum8(o, 64);
    if (lane < 8) part[summed8_index()] = f;
}

// MAXW: waves at most (four leave a wave the registers of a whole SIMD).
template <int MAXW>
__global__ void __launch_bounds__(64 * MAXW, 1) small_run_kernel(SmallRunArgs r)
{
    __shared__ Rec s_rec[kMaxSlots];
    __shared__ double s_part[kMaxSlots][MAXW][8];
    __shared__ int64_t s_min[MAXW];
    __shared__ int32_t s_cnt[MAXW];
    __shared__ int32_t s_stop;
    __shared__ int32_t s_hist[33];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.x;
    const int n = (int)r.n;
    const double tick = ldexp(1.0, -r.tick_bits);

    // this lane's particles: j = 256 wave + 64 k + lane; past the end
    // massless ones far away, never due
    double x[kPer][3], v[kPer][3], a[kPer][3], jk[kPer][3], m[kPer];
    int64_t t[kPer], dt[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int j = kTJ * wave + 64 * k + lane;
        const bool ok = j < n;
        const int q = ok ? j : 0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            x[k][d] = ok ? r.x[d * (int64_t)n + q] : 1.0e30;
            v[k][d] = ok ? r.v[d * (int64_t)n + q] : 0.0;
            a[k][d] = ok ? r.a[d * (int64_t)n + q] : 0.0;
            jk[k][d] = ok ? r.j[d * (int64_t)n + q] : 0.0;
        }
        m[k] = ok ? r.m[q] : 0.0;
        t[k] = ok ? r.t[q] : 0;
        dt[k] = ok ? r.dt[q] : 0;
    }
    if (tid < 33) s_hist[tid] = 0;
    if (tid < MAXW) {
        s_min[tid] = INT64_MAX;
        s_cnt[tid] = 0;
    }
    if (tid == 0) s_stop = 0;
    for (int q = tid; q < kMaxSlots * MAXW * 8; q += (int)blockDim.x)
        (&s_part[0][0][0])[q] = 0.0;
    __syncthreads();
    int64_t T = 0, inter = 0, done_steps = 0, last_T = 0;
    int32_t na = 0, last_na = 0, clamped = 0, bad = 0, heavy = 0, left = 0;
    bool gave_up = false;

    for (int64_t step = 1; step <= r.steps; ++step) {
        // ---- the block: T = min (t + dt), its particles in wave order -------
        int64_t e[kPer], mn = INT64_MAX;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const bool ok = kTJ * wave + 64 * k + lane < n;
            e[k] = ok ? t[k] + dt[k] : INT64_MAX;
            mn = min_i64(mn, e[k]);
        }
        mn = wave_min_i64(mn);
        // every wave's earliest time and how many of its particles have it:
        // where that is the block time, they are its part of the block
        bool act[kPer];
        unsigned long long due[kPer];
        int32_t c = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            act[k] = e[k] == mn && kTJ * wave + 64 * k + lane < n;
            due[k] = __ballot(act[k]);
            c += __popcll(due[k]);
        }
        if (lane == 0) {
            s_min[wave] = mn;
            s_cnt[wave] = c;
        }
        __syncthreads();
        T = s_min[0];
#pragma unroll
        for (int w = 1; w < MAXW; ++w) T = min_i64(T, s_min[w]);
        if (T > r.T_end) {
            na = 0;
            break;
        }
        int32_t base = 0;
        na = 0;
#pragma unroll
        for (int w = 0; w < MAXW; ++w) {
            const int32_t cw = s_min[w] == T ? s_cnt[w] : 0;
            base += w < wave ? cw : 0;
            na += cw;
        }
        const bool in_block = mn == T;   // this wave has particles in the block
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            act[k] = act[k] && in_block;
            due[k] = in_block ? due[k] : 0ull;
        }
        // ---- prediction, and this workgroup's active particles --------------
        int32_t pos[kPer];
        double px[kPer][3], pv[kPer][3];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            pos[k] = base + __popcll(due[k] & ((1ull << lane) - 1ull));
            base += __popcll(due[k]);
            OldState o;
            o.i = kTJ * wave + 64 * k + lane;
            o.t = t[k];
            o.dt = dt[k];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                o.x[d] = x[k][d];
                o.v[d] = v[k][d];
                o.a[d] = a[k][d];
                o.j[d] = jk[k][d];
            }
            predict_old(o, T, tick, px[k], pv[k]);
            if (act[k] && (pos[k] & (kSmallRunGrid - 1)) == g) {
                Rec& q = s_rec[pos[k] / kSmallRunGrid];
                q.o = o;
                q.pos = pos[k];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    q.xp[d] = px[k][d];
                    q.vp[d] = pv[k][d];
                }
            }
        }
        __syncthreads();
        // ---- the sweep: every wave its tile ----------------------------------
        const int mine = na > g ? (na - 1 - g) / kSmallRunGrid + 1 : 0;
        for (int s = 0; s < mine; ++s)
            sweep_slot(s_rec[s], px, pv, m, wave, r.eps2, s_part[s][wave]);
        __syncthreads();
        // ---- correct, publish, wait: the first wave ---------------------------
        double* buf = r.xbuf + (step & 1) * (int64_t)n * kSmallRunRec;
        if (wave == 0) {
            // a quad of lanes a particle, a lane a component (the fourth:
            // the potential), then a norm each
            for (int s0 = 0; s0 < mine; s0 += 16) {
                const int s = s0 + (lane >> 2), d = lane & 3;
                const bool ok = s < mine;
                const Rec& q = s_rec[ok ? s : 0];
                const int dd = d < 3 ? d : 0;
                double f0 = 0.0, f1 = 0.0;
#pragma unroll
                for (int w = 0; w < MAXW; ++w) {   // rows of absent waves are zero
                    f0 += s_part[ok ? s : 0][w][d < 3 ? d : 6];
                    f1 += s_part[ok ? s : 0][w][3 + dd];
                }
                const StepPowers sp = step_powers(q.o.dt, tick);
                double x1, v1, s1, c1;
                correct_component(sp, q.o.a[dd], q.o.j[dd], f0, f1, q.xp[dd], q.vp[dd], &x1, &v1,
                                  &s1, &c1);
                // lane d of the quad: the norm of acc, jerk, snap, crackle
                double u[3];
#pragma unroll
                for (int e1 = 0; e1 < 3; ++e1) {
                    const double ua = quad_value(f0, e1), uj = quad_value(f1, e1);
                    const double us = quad_value(s1, e1), uc = quad_value(c1, e1);
                    u[e1] = d == 0 ? ua : d == 1 ? uj : d == 2 ? us : uc;
                }
                const double nm = norm3(u[0], u[1], u[2]);
                const double crit = step_criterion(quad_value(nm, 0), quad_value(nm, 1),
                                                   quad_value(nm, 2), quad_value(nm, 3), r.eta,
                                                   r.form);
                int cl;
                const int64_t dn = quantize_dt(crit, r.tick_bits - log2_step(q.o.dt), T,
                                               r.tick_bits, r.k_min, r.k_max, &cl);
                if (ok) {
                    double* b = buf + (int64_t)q.pos * kSmallRunRec;
                    if (d < 3) {
                        put(b + d, x1);
                        put(b + 3 + d, v1);
                        put(b + 6 + d, f0);
                        put(b + 9 + d, f1);
                    } else {
                        put(b + 12, __longlong_as_double((long long)dn));
                        put(r.pot + q.o.i, f0);
                        clamped += cl;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");   // the records are written
            if (lane == 0)
                __hip_atomic_store(&r.flags[g * kSmallRunLine], r.epoch + step, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            if (!wait_all(r.flags, r.epoch + step, step == 1 ? r.arrival : r.patience, r.launch) &&
                lane == 0)
                s_stop = 1;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        if (s_stop) {
            gave_up = true;
            break;
        }
        // ---- take every corrected particle -------------------------------------
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            if (act[k]) {
                const double* b = buf + (int64_t)pos[k] * kSmallRunRec;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    x[k][d] = get(b + d);
                    v[k][d] = get(b + 3 + d);
                    a[k][d] = get(b + 6 + d);
                    jk[k][d] = get(b + 9 + d);
                }
                dt[k] = __double_as_longlong(get(b + 12));
                t[k] = T;
            }
        }
        inter += (int64_t)na * n;
        ++done_steps;
        last_T = T;
        last_na = na;
        if (g == 0 && tid == 0) s_hist[32 - __clz(na)] += 1;
        if (step % r.check_every == 0 && step < r.steps) {
            bad = __syncthreads_or(non_finite(x, v, a, jk) ? 1 : 0);
            if (bad) break;
        }
        heavy = (int64_t)na * n > kSmallRunHeavy ? heavy + 1 : 0;
        if (heavy == kSmallRunHeavyRow && step < r.steps) {
            left = 1;
            break;
        }
    }
    if (!gave_up && !bad) bad = __syncthreads_or(non_finite(x, v, a, jk) ? 1 : 0);

    // ---- does the launch count? -------------------------------------------------
    if (wave == 0) {
        bool ok = !gave_up;
        if (ok) {
            if (lane == 0)
                __hip_atomic_store(&r.flags[g * kSmallRunLine], r.epoch + r.steps + 1,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok = wait_all(r.flags, r.epoch + r.steps + 1, r.patience, r.launch);
        }
        if (lane == 0) s_stop = settle(&r.flags[kSmallRunGrid * kSmallRunLine], r.launch, ok) ? 0 : 1;
    }
    __syncthreads();
    const bool commit = s_stop == 0;
    if (commit) {
        // each chunk of 64 particles by one workgroup (all hold the same)
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int j = kTJ * wave + 64 * k + lane;
            if (j < n && done_steps > 0 && kPer * wave + k == g) {
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
        if (wave == 0) {
            const int32_t cl = wave_sum_i32(clamped);
            if (lane == 0 && cl > 0)
                atomicAdd((unsigned long long*)&r.counters[2], (unsigned long long)cl);
        }
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
        h->left = left;
        h->launch = r.launch;
    }
}

}  // namespace

bool small_run_plans(const SweepArgs& a)
{
    if (a.n_clusters != 1 || a.n > kSmallRunMax) return false;
    // every block's plan: 64 lanes a particle, chunks of one tile
    for (int32_t na = 1; na <= (int32_t)a.n; ++na) {
        int32_t L, ti;
        int64_t jc;
        plan_split(a, na, 1, &L, &ti, &jc);
        if (L != 64 || jc != kTJ) return false;
    }
    return true;
}

hipError_t launch_small_run(const SmallRunArgs& r, hipStream_t st)
{
    const int waves = (int)((r.n + kTJ - 1) / kTJ);
    if (waves <= 4)
        hipLaunchKernelGGL(small_run_kernel<4>, dim3(kSmallRunGrid), dim3(64 * waves), 0, st, r);
    else
        hipLaunchKernelGGL(small_run_kernel<6>, dim3(kSmallRunGrid), dim3(64 * waves), 0, st, r);
    return hipGetLastError();
}

}  // namespace hm
