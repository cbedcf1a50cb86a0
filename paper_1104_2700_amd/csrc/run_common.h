// Parts shared by the kernels that stay on the chip for many block steps.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hm {

// Relaxed device-scope accesses: past the per-XCD L2s, in no order.
__device__ __forceinline__ void put(double* p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get(const double* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int64_t get(const int64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Lane e of the lane's quad.
__device__ __forceinline__ double quad_value(double v, int e)
{
    const long long b = __double_as_longlong(v);
    int lo = (int)b, hi = (int)(b >> 32);
    switch (e) {
    case 0:
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x00, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x00, 0xF, 0xF, false);
        break;
    case 1:
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x55, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x55, 0xF, 0xF, false);
        break;
    case 2:
        lo = __builtin_amdgcn_update_dpp(0, lo, 0xAA, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0xAA, 0xF, 0xF, false);
        break;
    default:
        lo = __builtin_amdgcn_update_dpp(0, lo, 0xFF, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0xFF, 0xF, 0xF, false);
    }
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// Whether a workgroup has given the launch up (who waits for it then does too).
__device__ __forceinline__ bool given_up(const int64_t* verdict, int64_t launch)
{
    return get(verdict) == 2 * launch + 1;
}

// The launch's verdict: the first word set for it stands.
__device__ inline bool settle(int64_t* verdict, int64_t launch, bool commit)
{
    const unsigned long long mine = 2ull * (unsigned long long)launch + (commit ? 0ull : 1ull);
    unsigned long long old = (unsigned long long)get(verdict);
    while (old < 2ull * (unsigned long long)launch) {
        const unsigned long long seen = atomicCAS((unsigned long long*)verdict, old, mine);
        if (seen == old) return commit;
        old = seen;
    }
    return old == 2ull * (unsigned long long)launch;
}

// As hermite_check_finite: the launch checks the state where the host would
// have, after every check_every steps and at its end.
template <int K>
__device__ __forceinline__ bool non_finite(const double (&x)[K][3], const double (&v)[K][3],
                                           const double (&a)[K][3], const double (&j)[K][3])
{
    bool bad = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
        for (int d = 0; d < 3; ++d)
            bad = bad || !__builtin_isfinite(x[k][d]) || !__builtin_isfinite(v[k][d]) ||
                  !__builtin_isfinite(a[k][d]) || !__builtin_isfinite(j[k][d]);
    }
    return bad;
}

}  // namespace hm
