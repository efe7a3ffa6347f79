// Chains of dependent fmas over values in LDS (gfx950).
//
// The sequential order of the updates is part of the result, so these sums stay
// one fma after another; what they must not wait for is an LDS round trip per
// few of them.  The next values are requested before the current ones are used,
// and keep_loads_above() holds the compiler to that (left alone it moves the
// requests down to their use, which costs the round trip again).  Arrays are
// padded to whole steps with +0: fma(-0, +0, acc) adds -0, which changes no acc.
#pragma once

#include <hip/hip_runtime.h>

namespace kcdev {

// Wave-local LDS ordering: every lane's LDS writes are visible to the other
// lanes of the same wavefront after this point.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void keep_loads_above() { asm volatile("" ::: "memory"); }

// Entries of a chain are padded to a multiple of this.
constexpr int kChainPad = 16;
__host__ __device__ constexpr int chain_padded(int n) { return (n + kChainPad - 1) / kChainPad * kChainPad; }

// acc <- fma(-v, v, acc) over the staged row of np values in ascending order, in FP64 (padded, see pad_row).
template <typename VT>
__device__ __forceinline__ double pivot_sum(const VT* __restrict__ sval, int np, double acc) {
    typedef VT vec __attribute__((ext_vector_type(16 / sizeof(VT))));
    constexpr int kPer = 16 / sizeof(VT), kVec = 8 / kPer;
    struct Eight {
        vec v[kVec];
    };
    const vec* v = reinterpret_cast<const vec*>(sval);
    auto load = [&](Eight& e, int q) {
#pragma unroll
        for (int u = 0; u < kVec; ++u) e.v[u] = v[q / kPer + u];
    };
    auto apply = [&](const Eight& e) {
#pragma unroll
        for (int u = 0; u < kVec; ++u)
#pragma unroll
            for (int w = 0; w < kPer; ++w) {
                const double x = double(e.v[u][w]);
                acc = __builtin_fma(-x, x, acc);
            }
    };
    if (np <= 0) return acc;
    Eight a, b;
    load(a, 0);
    for (int t = 0; t < np; t += 16) {
        load(b, t + 8);
        keep_loads_above();
        apply(a);
        load(a, t + 16 < np ? t + 16 : 0);
        keep_loads_above();
        apply(b);
    }
    return acc;
}

// Pads a staged row of np values for pivot_sum.
template <typename VT>
__device__ __forceinline__ void pad_row(VT* sval, int np, int tid) {
    if (tid < chain_padded(np) - np) sval[np + tid] = VT(0);
}

}  // namespace kcdev
