// The FP64 pair term shared by the sweeps.
#pragma once

#include <hip/hip_runtime.h>

namespace hm {

__device__ __forceinline__ double rsqrt_f64(double s)
{
    // y0 from the hardware; with e = 1 - s y0^2,
    // 1/sqrt(s) = y0 (1 - e)^{-1/2} = y0 (1 + e/2 + 3 e^2 / 8 + ...).
    const double y = __builtin_amdgcn_rsq(s);
    const double h = s * y;
    const double e = fma(-h, y, 1.0);
    const double p = fma(e, 0.375, 0.5);
    return fma(y * e, p, y);
}

struct I64 {   // i-particle in FP64
    double x, y, z, vx, vy, vz;
};

struct SumD {  // FP64 sums: acc, jerk, sum of m/r; FP32 error estimates
    double ax, ay, az, jx, jy, jz, pp;
    float ea, ej;  // sums over FP32 runs of |run sum|^2 (acc, jerk)
    __device__ __forceinline__ void zero()
    {
        ax = ay = az = jx = jy = jz = pp = 0.0;
        ea = ej = 0.0f;
    }
    __device__ __forceinline__ void add(const SumD& o)
    {
        ax += o.ax; ay += o.ay; az += o.az;
        jx += o.jx; jy += o.jy; jz += o.jz;
        pp += o.pp;
    }
};

// One FP64 pair term: with b3 = 3 (r.v) / s,
//   acc += m/s^{3/2} r,  jerk += m/s^{3/2} (v - b3 r),  pp += m/s^{1/2}.
template <bool MASK>
__device__ __forceinline__ void pair_f64(const I64& I, double eps2, double xj,
                                         double yj, double zj, double vxj,
                                         double vyj, double vzj, double mj,
                                         bool self, SumD& S)
{
    const double dx = xj - I.x, dy = yj - I.y, dz = zj - I.z;
    const double dvx = vxj - I.vx, dvy = vyj - I.vy, dvz = vzj - I.vz;
    const double r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, eps2)));
    double ri = rsqrt_f64(r2);
    if (MASK) ri = self ? 0.0 : ri;
    const double mr = mj * ri;
    const double ri2 = ri * ri;
    const double mr3 = mr * ri2;
    const double rv = fma(dx, dvx, fma(dy, dvy, dz * dvz));
    const double b3 = (rv * ri2) * 3.0;
    S.pp = fma(mj, ri, S.pp);
    S.ax = fma(mr3, dx, S.ax);
    S.ay = fma(mr3, dy, S.ay);
    S.az = fma(mr3, dz, S.az);
    S.jx = fma(mr3, fma(-b3, dx, dvx), S.jx);
    S.jy = fma(mr3, fma(-b3, dy, dvy), S.jy);
    S.jz = fma(mr3, fma(-b3, dz, dvz), S.jz);
}

}  // namespace hm
