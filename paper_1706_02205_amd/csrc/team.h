// The factorization of one DAG level by teams of wavefronts (team.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "factor.h"

namespace kc {

// LDS of a team workgroup for rows of at most max_row parents and columns up to max_col.
size_t team_lds(int32_t max_row, int32_t max_col, size_t value_bytes);

// Block units [ub, ue) (64 entries of a column each, columns up to max_col) of one level.
template <typename VT>
hipError_t launch_team(const kc_factor* f, bool count, int policy, double tau, int64_t ub, int64_t ue,
                       int32_t max_col, hipStream_t s);

// The same, and in the same launch the forward sweep (all nrhs right-hand sides) of
// rows [rb, re) of fwd_rows, a level before it; either may be empty.
template <typename VT>
hipError_t launch_team_fwd(const kc_factor* f, int policy, double tau, int64_t ub, int64_t ue, int32_t max_col,
                           const double* b, double* y, int nrhs, int64_t rb, int64_t re, hipStream_t s);

}  // namespace kc
