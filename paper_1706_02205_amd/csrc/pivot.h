// The pivot's sum of squares in sequence (gfx950).
#pragma once

#include <hip/hip_runtime.h>

namespace kcdev {

constexpr int kPivotStep = 16;

// Entries of LDS that a staged row of np parents takes: the sum below reads whole
// steps, and what it reads past the row must be +0 (pad_row).
__host__ __device__ constexpr int pivot_padded(int np) { return (np + kPivotStep - 1) / kPivotStep * kPivotStep; }

template <typename VT>
__device__ __forceinline__ void pad_row(VT* sval, int np, int tid) {
    if (tid < pivot_padded(np) - np) sval[np + tid] = VT(0);
}

// acc <- fma(-v, v, acc) over the staged row in ascending order, in FP64.  The
// chain of dependent fmas is short (8 cycles each); what made this loop long is an
// LDS round trip per value or two, so 16 values are read at once and the next 16
// requested before the current ones are used.  The padding's fma(-0, +0, acc)
// adds -0, which changes no acc.
template <typename VT>
__device__ __forceinline__ double pivot_sum(const VT* __restrict__ sval, int np, double acc) {
    typedef VT vec __attribute__((ext_vector_type(16 / sizeof(VT))));
    constexpr int kPer = 16 / sizeof(VT), kVec = kPivotStep / kPer;
    const vec* v = reinterpret_cast<const vec*>(sval);
    vec cur[kVec];
    if (np > 0) {
#pragma unroll
        for (int u = 0; u < kVec; ++u) cur[u] = v[u];
    }
    for (int t = 0; t < np; t += kPivotStep) {
        vec nxt[kVec];
        const int at = t + kPivotStep < np ? (t + kPivotStep) / kPer : 0;
#pragma unroll
        for (int u = 0; u < kVec; ++u) nxt[u] = v[at + u];
#pragma unroll
        for (int u = 0; u < kVec; ++u)
#pragma unroll
            for (int w = 0; w < kPer; ++w) {
                const double x = double(cur[u][w]);
                acc = __builtin_fma(-x, x, acc);
            }
#pragma unroll
        for (int u = 0; u < kVec; ++u) cur[u] = nxt[u];
    }
    return acc;
}

}  // namespace kcdev
