// The forward sweep and the backward sweep's small levels (gfx950): a workgroup per
// row where a level has few, a wavefront per row in large forward levels.
//
// The sequential substitution of a row is a chain of fmas, one per entry, over
// values that arrive through two dependent loads (the index, then the gathered
// right-hand-side row).  In a level of few rows nothing hides those: a wavefront
// per row took 384 entries at a time (bwd_solve still does, in large levels), and
// each such step waited for both loads and then for an LDS round trip per eight
// fmas.  Here the four wavefronts of a workgroup gather a block of the row while
// the first (and, past four right-hand sides, the second) runs the previous
// block's chains, 16 lanes to a right-hand side (row_chain.h).  Measured, a whole
// solve: 2,000 points 1.33 -> 0.94 ms, 20,011 in 3-D 5.6 -> 3.9 ms, 90,601 grid
// points with 8 right-hand sides 6.8 -> 4.8 ms, 160,000 with one 5.9 -> 4.3 ms; with the
// schedules' row pointers and long columns summed across a workgroup 0.72, 3.15,
// 3.8 and 3.6 ms.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "sweep.h"
#include "sweep_dev.h"

using namespace kcdev;

namespace {

constexpr int kThreads = 256;

// The first nsum rows are columns summed across the workgroup (backward only, instances with a sound factor).
template <typename VT, int NR, bool FWD>
__global__ __launch_bounds__(kThreads) void sweep_narrow(SweepArgs<VT> a, int64_t beg, int nsum) {
    __shared__ __align__(16) double lds[sweep_lds(NR, kThreads)];
    kc::SweepRow row = a.rows[beg + int64_t(blockIdx.x)];
    if constexpr (!FWD) {
        const bool unsound = row.n < 0;
        row.n = max(row.n, ~row.n);
        if (int(blockIdx.x) < nsum && !unsound) {
            sum_column<VT, NR>(a, row, lds);
            return;
        }
    }
    sweep_row<VT, NR, kThreads, FWD>(a, row, NR, lds);
}

// Rows of a large level, a wavefront each; every XCD takes one contiguous range.
template <typename VT, int NR>
__global__ __launch_bounds__(kThreads) void fwd_wide(SweepArgs<VT> a, int64_t beg, int64_t end) {
    const int64_t t = beg + int64_t(xcd_block()) * (kThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    if (t < end) wide_row<VT, NR>(a, a.rows[t], threadIdx.x % 64);
}

template <typename VT, bool FWD>
hipError_t launch(const SweepArgs<VT>& a, int nr, int64_t beg, int64_t end, int64_t sums, hipStream_t s) {
    if (end <= beg) return hipSuccess;
    auto go = [&](auto w) {
        constexpr int NR = decltype(w)::value;
        if constexpr (FWD) {
            if (end - beg >= kWideRows) {
                fwd_wide<VT, NR><<<unsigned((end - beg + 3) / 4), kThreads, 0, s>>>(a, beg, end);
                return;
            }
        }
        sweep_narrow<VT, NR, FWD><<<unsigned(end - beg), kThreads, 0, s>>>(a, beg, int(sums - beg));
    };
    switch (nr) {
        case 1: go(std::integral_constant<int, 1>()); break;
        case 2: go(std::integral_constant<int, 2>()); break;
        case 3: go(std::integral_constant<int, 3>()); break;
        case 4: go(std::integral_constant<int, 4>()); break;
        case 5: go(std::integral_constant<int, 5>()); break;
        case 6: go(std::integral_constant<int, 6>()); break;
        case 7: go(std::integral_constant<int, 7>()); break;
        default: go(std::integral_constant<int, 8>()); break;
    }
    return hipGetLastError();
}

}  // namespace

namespace kc {

template <typename VT>
hipError_t launch_fwd(const kc_factor* f, const double* b, int ld, int r0, int nr, double* y, int64_t rb,
                             int64_t re, hipStream_t s) {
    return launch<VT, true>(fwd_args<VT>(f, b, ld, r0, y), nr, rb, re, rb, s);
}

template <typename VT>
hipError_t launch_bwd_narrow(const kc_factor* f, double* x, int ld, int r0, int nr, double* y, int64_t cb, int64_t ce,
                             int64_t cm, hipStream_t s) {
    const SweepArgs<VT> a{f->bwd_desc, f->rowidx, static_cast<const VT*>(f->Lcsc), f->diag, nullptr, x, y, ld, r0};
    return launch<VT, false>(a, nr, cb, ce, cm, s);
}

template hipError_t launch_fwd<double>(const kc_factor*, const double*, int, int, int, double*, int64_t, int64_t,
                                              hipStream_t);
template hipError_t launch_fwd<float>(const kc_factor*, const double*, int, int, int, double*, int64_t, int64_t,
                                             hipStream_t);
template hipError_t launch_bwd_narrow<double>(const kc_factor*, double*, int, int, int, double*, int64_t, int64_t,
                                              int64_t, hipStream_t);
template hipError_t launch_bwd_narrow<float>(const kc_factor*, double*, int, int, int, double*, int64_t, int64_t,
                                             int64_t, hipStream_t);

}  // namespace kc
