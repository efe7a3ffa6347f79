// The factorization of one DAG level by teams of wavefronts (team.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "factor.h"

namespace kc {

// LDS of a team workgroup for rows of at most max_row parents and columns up to max_col.
size_t team_lds(int32_t max_row, int32_t max_col, size_t value_bytes);

// One level's units.
template <typename VT>
hipError_t launch_team(const kc_factor* f, bool count, int policy, double tau, int level, hipStream_t s);

// The same (none for level = the number of levels), and in the same launch the
// forward sweep, all nrhs right-hand sides, of rows [rb, re) of an earlier level.
template <typename VT>
hipError_t launch_team_fwd(const kc_factor* f, int policy, double tau, int level, const double* b, double* y, int nrhs,
                           int64_t rb, int64_t re, hipStream_t s);

}  // namespace kc
