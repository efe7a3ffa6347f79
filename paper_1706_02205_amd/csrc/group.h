// The factorization by supernodal groups on the matrix cores (group.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "factor.h"

namespace kc {

constexpr int kGroupCols = 16;  // columns of a group: the width of the MFMA tile
constexpr int kGroupRows = 48;  // panel rows of a unit, beside the group's 16 diagonal rows

// Units [ub, ue) of one level of the group DAG; twonu = 2 nu.
hipError_t launch_group(const kc_factor* f, int twonu, double ell, int policy, double tau, int64_t ub, int64_t ue,
                        hipStream_t s);

}  // namespace kc
