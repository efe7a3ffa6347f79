// Device code of the triangular sweeps, shared by the kernels that run rows of
// them (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include "factor.h"
#include "row_chain.h"

namespace kcdev {

// Workgroups are dealt to the 8 XCDs round-robin (block b runs on XCD b % 8).
// Renumber them so that each XCD receives one contiguous range of blocks: the
// rows and columns of a solve level are laid out in spatial order, so each
// XCD's L2 then serves one region of the point cloud.  (The factorization's
// units are ordered by length instead, and keep the plain block order.)
constexpr int kNumXcd = 8;
__device__ __forceinline__ int xcd_block() {
    const int b = blockIdx.x, nb = gridDim.x;
    const int q = nb / kNumXcd, r = nb % kNumXcd;
    const int x = b % kNumXcd, i = b / kNumXcd;
    return x * q + (x < r ? x : r) + i;
}

template <typename VT>
__device__ __forceinline__ double diag_value(const VT* Lv, const double* diag, int64_t pos, int k) {
    if constexpr (sizeof(VT) == 8) return Lv[pos];
    else return diag[k];
}

// s[r] += sum of L_e * y[row_e][r] over this lane's entries e = e, e + STRIDE,
// ... below e1, in ascending order: four entries in flight at once, and the row
// indices of the next four requested before this four's values and gathers,
// so each step waits for one round trip instead of two.
template <typename VT, int NR, int STRIDE = 64>
__device__ __forceinline__ void dot_entries(const int32_t* __restrict__ rowidx, const VT* __restrict__ Lcsc, int64_t e,
                                            int64_t e1, const double* __restrict__ y, int ld, int r0,
                                            double (&s)[NR]) {
    constexpr int kDepth = 4;
    int ci[kDepth];
#pragma unroll
    for (int u = 0; u < kDepth; ++u) {
        const int64_t eu = e + int64_t(u) * STRIDE;
        ci[u] = eu < e1 ? rowidx[eu] : -1;
    }
    for (; e < e1; e += kDepth * STRIDE) {
        int cn[kDepth];
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            const int64_t en = e + int64_t(kDepth + u) * STRIDE;
            cn[u] = en < e1 ? rowidx[en] : -1;
        }
        double l[kDepth], v[kDepth][NR];
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            l[u] = 0.0;
            if (ci[u] >= 0) {
                l[u] = double(Lcsc[e + int64_t(u) * STRIDE]);
                const double* xk = y + int64_t(ci[u]) * ld + r0;
#pragma unroll
                for (int r = 0; r < NR; ++r) v[u][r] = xk[r];
            }
        }
#pragma unroll
        for (int u = 0; u < kDepth; ++u)
            if (ci[u] >= 0) {
#pragma unroll
                for (int r = 0; r < NR; ++r) s[r] = __builtin_fma(l[u], v[u][r], s[r]);
            }
#pragma unroll
        for (int u = 0; u < kDepth; ++u) ci[u] = cn[u];
    }
}

// Forward levels of at least kWideRows rows: there a wavefront's 64 lanes share
// a row's dot product (every 64th entry, four in flight) and a fixed butterfly
// adds them, instead of 8 lanes applying staged chunks in the sequential
// order -- more throughput on large levels and a shorter chain per row on
// medium ones.  Deterministic, but not the sequential substitution's
// summation order; smaller levels keep that order.
constexpr int64_t kWideRows = 1024;

template <typename VT, int NR>
__device__ __forceinline__ double wave_dot(const int32_t* __restrict__ idx, const VT* __restrict__ val, int64_t b0,
                                           int64_t b1, const double* __restrict__ src, int ld, int r0, int lane) {
    double s[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) s[r] = 0.0;
    dot_entries<VT, NR>(idx, val, b0 + lane, b1, src, ld, r0, s);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s[r] += __shfl_xor(s[r], off, 64);
    double v = s[0];
#pragma unroll
    for (int r = 1; r < NR; ++r)
        if (lane == r) v = s[r];
    return v;  // lane r < NR holds right-hand side r's sum
}

constexpr int kMaxRhs = 8;  // right-hand sides of one pass over L

// What the two sweeps differ in: the rows' entries, where the right-hand side
// comes from and where x goes.
template <typename VT>
struct SweepArgs {
    const kc::SweepRow* rows;
    const int32_t* idx;
    const VT* val;
    const double* diag;
    const double* b;  // forward: right-hand side, original order
    double* x;        // backward: solution, original order
    double* y;
    int ld, r0;
};

template <typename VT>
SweepArgs<VT> fwd_args(const kc_factor* f, const double* b, int ld, int r0, double* y) {
    return {f->fwd_desc, f->colidx, static_cast<const VT*>(f->L), f->diag, b, nullptr, y, ld, r0};
}

// One row of a wide forward level by a wavefront.
template <typename VT, int NR>
__device__ __forceinline__ void wide_row(const SweepArgs<VT>& a, const kc::SweepRow row, int lane) {
    const int k = row.k;
    const int64_t p0 = row.p0, pd = p0 + row.n;  // pd: the diagonal
    const double v = wave_dot<VT, NR>(a.idx, a.val, p0, pd, a.y, a.ld, a.r0, lane);
    if (lane < NR) {
        const double lkk = diag_value(a.val, a.diag, pd, k);
        const double acc = a.b[int64_t(row.perm) * a.ld + a.r0 + lane] - v;
        a.y[int64_t(k) * a.ld + a.r0 + lane] = (lkk == 0.0) ? 0.0 : acc / lkk;
    }
}

// One row by a workgroup of THREADS (a multiple of 16), right-hand sides r0 ..
// r0 + nr - 1 (nr <= NR).  The chain is a row chain per right-hand side (L staged
// negated).  Entries past the row's end are staged as -0 and +0: fma(-0, +0, acc)
// changes no acc, so the result is the sequential substitution's bit for bit.
template <typename VT, int NR, int THREADS, bool FWD>
__device__ __forceinline__ void sweep_row(const SweepArgs<VT>& a, const kc::SweepRow row, int nr,
                                          double* __restrict__ lds) {
    constexpr int kStride = THREADS + 2;  // rows of consecutive right-hand sides 4 banks apart
    const int tid = threadIdx.x;
    auto sL = [&](int buf) { return lds + buf * THREADS; };
    auto sY = [&](int buf) { return lds + 2 * THREADS + buf * NR * kStride; };
    const int k = row.k, n = row.n;
    const int64_t p0 = row.p0, pd = FWD ? p0 + n : p0 - 1;  // pd: the diagonal
    int ci, cn;
    double lv, ln, v[NR];
    auto entries = [&](int at, int& c, double& l) {
        const int q = at + tid;
        c = q < n ? a.idx[p0 + q] : -1;
        l = q < n ? double(a.val[p0 + q]) : 0.0;
    };
    auto gather = [&]() {
        const double* src = a.y + int64_t(ci < 0 ? 0 : ci) * a.ld + a.r0;
#pragma unroll
        for (int r = 0; r < NR; ++r) v[r] = ci < 0 || r >= nr ? 0.0 : src[r];
    };
    auto stage = [&](int buf) {
        sL(buf)[tid] = -lv;
#pragma unroll
        for (int r = 0; r < NR; ++r) sY(buf)[r * kStride + tid] = v[r];
    };
    entries(0, ci, lv);
    entries(THREADS, cn, ln);
    // right-hand side r is the business of 16 lanes: rows 0 .. 3 of wavefront 0, then of wavefront 1
    const int r = tid / kRowLanes;
    const bool chains = tid < 64 * ((NR + 3) / 4);  // whole wavefronts
    double acc = 0.0, lkk = 1.0;
    if (r < nr) {
        acc = FWD ? a.b[int64_t(row.perm) * a.ld + a.r0 + r] : a.y[int64_t(k) * a.ld + a.r0 + r];
        lkk = diag_value(a.val, a.diag, pd, k);
    }
    if (n > 0) {
        gather();
        stage(0);
        __syncthreads();
        for (int at = 0; at < n; at += THREADS) {
            const int buf = (at / THREADS) & 1;
            const bool more = at + THREADS < n;
            if (more) {  // the next block's rows and the indices after it, in flight while the chain runs
                ci = cn;
                lv = ln;
                gather();
                entries(at + 2 * THREADS, cn, ln);
            }
            const int m = n - at < THREADS ? chain_padded(n - at) : THREADS;
            if (chains) acc = row_chain(sL(buf), sY(buf) + (r < NR ? r : 0) * kStride, m, acc);
            if (more) {
                stage(buf ^ 1);
                __syncthreads();
            }
        }
    }
    if (r < nr && tid % kRowLanes == 0) {
        const double x = lkk == 0.0 ? 0.0 : acc / lkk;
        a.y[int64_t(k) * a.ld + a.r0 + r] = x;
        if constexpr (!FWD) a.x[int64_t(row.perm) * a.ld + a.r0 + r] = x;
    }
}

// One backward column by a workgroup of 256: its threads take every 256th entry,
// each wavefront reduces by a fixed butterfly, and the wavefronts' sums are added in
// order.  Deterministic, but not the sequential substitution's order.
template <typename VT, int NR>
__device__ __forceinline__ void sum_column(const SweepArgs<VT>& a, const kc::SweepRow row, double* __restrict__ lds) {
    constexpr int kThreads = 256, kWaves = kThreads / 64;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int64_t p0 = row.p0;
    double* yk = a.y + int64_t(row.k) * a.ld + a.r0 + lane;
    double own = 0.0, lkk = 1.0;
    if (wave == 0 && lane < NR) {
        own = *yk;
        lkk = diag_value(a.val, a.diag, p0 - 1, row.k);
    }
    double s[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) s[r] = 0.0;
    dot_entries<VT, NR, kThreads>(a.idx, a.val, p0 + threadIdx.x, p0 + row.n, a.y, a.ld, a.r0, s);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s[r] += __shfl_xor(s[r], off, 64);
    if (lane < NR) {
        double v = s[0];
#pragma unroll
        for (int r = 1; r < NR; ++r)
            if (lane == r) v = s[r];
        lds[wave * NR + lane] = v;
    }
    __syncthreads();
    if (wave == 0 && lane < NR) {
        double v = lds[lane];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += lds[w * NR + lane];
        const double x = lkk == 0.0 ? 0.0 : (own - v) / lkk;
        *yk = x;
        a.x[int64_t(row.perm) * a.ld + a.r0 + lane] = x;
    }
}

// Doubles of LDS that sweep_row takes.
constexpr size_t sweep_lds(int nr, int threads) { return 2 * size_t(threads) + 2 * size_t(nr) * size_t(threads + 2); }

}  // namespace kcdev
