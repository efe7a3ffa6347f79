// The forward sweep and the backward sweep's small levels (sweep.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "factor.h"

namespace kc {

// Rows [rb, re) of fwd_desc, one level: y = (P b - L y) / L_kk for right-hand sides r0 .. r0 + nr - 1 (nr <= 8).
template <typename VT>
hipError_t launch_fwd(const kc_factor* f, const double* b, int ld, int r0, int nr, double* y, int64_t rb,
                             int64_t re, hipStream_t s);
// Columns [cb, ce) of bwd_short: x = (y - L^T x) / L_jj, into y and (original order)
// x.  Those before cm are summed across a workgroup if their instance's factor is
// sound, the others in sequence.
template <typename VT>
hipError_t launch_bwd_narrow(const kc_factor* f, double* x, int ld, int r0, int nr, double* y, int64_t cb, int64_t ce,
                             int64_t cm, hipStream_t s);

}  // namespace kc
