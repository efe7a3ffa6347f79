// Chains of dependent fmas over values held by the lanes of a row (gfx950).
//
// A wavefront is four rows of 16 lanes.  Lane s of a row holds the s-th pair (a, b)
// of the row's chain, and every lane of the row runs acc <- fma(a_n, b_n, acc) for
// n = 0 .. 15 in that order: row_newbcast hands lane n's values to the whole row,
// two vector instructions a step and no LDS: 12.5 cycles a step, measured, against
// 17.6 with the pairs read from LDS (a 128-bit read a step, whether one lane or 64
// use it) and 9.3 for the fma alone.  All 64 lanes must be active.  The leading s_nop keeps the two wait states
// that a broadcast needs after its source was written by a vector instruction.  The
// steps are aligned to their 8 bytes: where a change elsewhere in the kernel left
// them across 8-byte boundaries, a solve of 48 problems took 1.574 ms, not 1.530.
#pragma once

#include <hip/hip_runtime.h>

#include "chain.h"

namespace kcdev {

constexpr int kRowLanes = 16;

// The 16 steps in one block, so that nothing writes a source between the wait and a broadcast.
__device__ __forceinline__ void row_chain_steps(double& acc, double a, double b) {
    double t;
    asm volatile(
        "s_nop 1\n\t"
        ".p2align 3\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_mov_b64_dpp %1, %2 row_newbcast:15 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %0, %3, %1 row_newbcast:15 row_mask:0xf bank_mask:0xf\n\t"
        : "+v"(acc), "=&v"(t)
        : "v"(a), "v"(b));
}
// The 16 steps over entries 0 .. m - 1 (m a positive multiple of 16) of two arrays in
// LDS, the next step's values requested before the current one's fmas.
__device__ __forceinline__ double row_chain(const double* __restrict__ a, const double* __restrict__ b, int m,
                                            double acc) {
    const int s = threadIdx.x % kRowLanes;
    double av = a[s], bv = b[s];
    for (int t = 0; t < m; t += kRowLanes) {
        const int next = (t + kRowLanes < m ? t + kRowLanes : 0) + s;
        const double an = a[next], bn = b[next];
        keep_loads_above();
        row_chain_steps(acc, av, bv);
        av = an;
        bv = bn;
    }
    return acc;
}

}  // namespace kcdev
