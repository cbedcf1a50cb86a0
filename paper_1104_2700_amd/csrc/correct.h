// The corrector's arithmetic for one particle, shared by the corrector
// kernels and the small-system run.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hm {

__device__ __forceinline__ int log2_step(int64_t dt)
{
    return 63 - __clzll((unsigned long long)dt);
}

// ---- timestep: Aarseth criterion and power-of-two quantisation ----------
__device__ __forceinline__ double norm3(double a, double b, double c)
{
    return sqrt(fma(a, a, fma(b, b, c * c)));
}

__device__ inline int64_t quantize_dt(double crit, int k_old, int64_t T, int tick_bits,
                               int k_min, int k_max, int* clamped)
{
    int k;
    *clamped = 0;
    if (__builtin_isnan(crit) || __builtin_isinf(crit)) {
        k = k_min;
    } else if (crit <= 0.0) {
        k = k_max;
        *clamped = 1;
    } else {
        int e;
        frexp(crit, &e);            // crit in [2^(e-1), 2^e)
        k = 1 - e;
        if (k < k_min) k = k_min;
        if (k > k_max) { k = k_max; *clamped = 1; }
    }
    if (k_old >= 0 && k < k_old - 1) k = k_old - 1;
    // halved until the block time is a multiple of it
    if (k < k_max && T != 0) {
        const int kc = tick_bits - (int)__builtin_ctzll((unsigned long long)T);
        if (k < kc) k = kc < k_max ? kc : k_max;
    }
    return ((int64_t)1) << (tick_bits - k);
}

// The pre-step state of an active particle that the corrector reads, loaded
// before the new forces are summed so that these loads overlap the sum's.
struct OldState {
    int i;                      // particle index
    int64_t t, dt;
    double x[3], v[3];          // x, v (prediction in place) or xp, vp
    double a[3], j[3];
};

// Equations (xpred), (vpred) for this particle, dt = T - t_i.
__device__ __forceinline__ void predict_old(const OldState& o, int64_t T, double tick,
                                            double xp[3], double vp[3])
{
    const double hp = (double)(T - o.t) * tick;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double ac = o.a[d], jk = o.j[d];
        xp[d] = fma(hp, fma(hp, fma(hp, jk * (1.0 / 6.0), ac * 0.5), o.v[d]), o.x[d]);
        vp[d] = fma(hp, fma(hp, jk * 0.5, ac), o.v[d]);
    }
}

struct Corrected {
    double x[3], v[3];
    double crit;
    int64_t dt;
    int clamped;
};

// x / y from r = 1 / y rounded to nearest: one correction of the product
// (Markstein's division step; exact where y is a power of two, as the steps
// of the block scheme are).  3 instructions for a division's 11.
__device__ __forceinline__ double div_by(double x, double y, double r)
{
    const double q = x * r;
    return fma(fma(-q, y, x), r, q);
}

// The powers of a particle's step that the corrector divides and multiplies by.
struct StepPowers {
    double h, h2, h3, h4, h5, r2, r3;
};

__device__ __forceinline__ StepPowers step_powers(int64_t dt_old, double tick)
{
    StepPowers s;
    s.h = (double)dt_old * tick;
    s.h2 = s.h * s.h;
    s.h3 = s.h2 * s.h;
    s.h4 = s.h3 * s.h;
    s.h5 = s.h4 * s.h;
    s.r2 = 1.0 / s.h2;
    s.r3 = 1.0 / s.h3;
    return s;
}

// One component: snap s0 and crackle c0 from the old and new force, the
// corrected position and velocity, the snap at the new time.  (Every
// rounding is written out, so that each kernel gives the same bits.)
__device__ __forceinline__ void correct_component(const StepPowers& p, double a0, double j0,
                                                  double a1, double j1, double xp, double vp,
                                                  double* x, double* v, double* s1, double* c)
{
#pragma clang fp contract(off)
    const double da = a0 - a1;
    const double s0 = div_by(2.0 * fma(-3.0, da, -(fma(2.0, j0, j1) * p.h)), p.h2, p.r2);
    const double c0 = div_by(6.0 * fma(2.0, da, (j0 + j1) * p.h), p.h3, p.r3);
    *x = xp + div_by(s0 * p.h4, 24.0, 1.0 / 24.0) + div_by(c0 * p.h5, 120.0, 1.0 / 120.0);
    *v = vp + div_by(s0 * p.h3, 6.0, 1.0 / 6.0) + div_by(c0 * p.h4, 24.0, 1.0 / 24.0);
    *s1 = fma(c0, p.h, s0);
    *c = c0;
}

// The criterion from the norms of the new acceleration, jerk, snap, crackle.
__device__ __forceinline__ double step_criterion(double A, double J, double S, double C,
                                                 double eta, int form)
{
#pragma clang fp contract(off)
    const double R = fma(A, S, J * J) / fma(J, C, S * S);
    return form == 0 ? eta * sqrt(R) : sqrt(eta * R);
}

// Steps 5-8 for a particle predicted at xp, vp: snap and crackle from the
// old and new force, the corrected x and v, and the next step.
__device__ __forceinline__ void correct_core(const OldState& o, const double xp[3],
                                             const double vp[3], int64_t T, double tick,
                                             int tick_bits, const double a1v[3],
                                             const double j1v[3], double eta, int form,
                                             int k_min, int k_max, Corrected* r)
{
    const StepPowers p = step_powers(o.dt, tick);
    double s1[3], cc[3];
#pragma unroll
    for (int d = 0; d < 3; ++d)
        correct_component(p, o.a[d], o.j[d], a1v[d], j1v[d], xp[d], vp[d], &r->x[d], &r->v[d],
                          &s1[d], &cc[d]);
    r->crit = step_criterion(norm3(a1v[0], a1v[1], a1v[2]), norm3(j1v[0], j1v[1], j1v[2]),
                             norm3(s1[0], s1[1], s1[2]), norm3(cc[0], cc[1], cc[2]), eta, form);
    const int k_old = tick_bits - log2_step(o.dt);
    r->dt = quantize_dt(r->crit, k_old, T, tick_bits, k_min, k_max, &r->clamped);
}

}  // namespace hm
