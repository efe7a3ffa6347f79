// ICHOL(0) by supernodal groups (gfx950).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "chain.h"
#include "crmath.h"
#include "group.h"

using namespace kc::counter;
using kc::kGroupCols;
using kc::kGroupRows;

namespace {

constexpr int kWave = 64;

// Supernodal groups on the matrix cores (mixed precision, supernodal plans).
//
// The block-closed pattern makes every member of a supernode J = [s0, s1) share
// one row structure: row g of a member is P(J) (the parents of s0), then s0..g-1;
// column g is g..s1-1, then the rows O_J of the other supernodes below J.  A
// group G = [g0, g1) of at most 16 consecutive members therefore shares its
// parents P_G = row g0 before its diagonal, and for a row k of column g0 the
// Schur updates of all 16 entries (k, g), g in G, run over the same parents
// i in P_G that row k holds:
//     a_kg = Theta_kg - sum_{i in P_G, i in row k} L_ki L_gi - sum_{g0 <= h < g} L_kh L_gh.
// The first sum, for 64 rows at once, is a dense product (64 x |P_G|) . (|P_G| x 16)
// on v_mfma_f32_16x16x4f32: row k's values are scattered into an LDS tile over
// P_G (row k is walked once for the whole group, instead of once per column as
// in the element-wise kernel) and the group's rows L_{G,P_G} form the other
// operand.  The second sum and the divisions follow in registers, column by
// column: the dense Cholesky of the group's diagonal block with FP64 pivots
// (accumulated as in the element-wise kernel, FP32 x FP32 products exact in
// FP64), then the panel rows.  A unit is one group with its 16 diagonal rows
// (recomputed by every unit of the group, written by the first) and 48 panel
// rows; the units of a level of the group DAG run in one launch.
//
// The product itself is short (a busy matrix core 1% of the time when a
// wavefront did all of a unit's work: 471 us a level at 10,007 points); the walks
// are what takes time.  So a workgroup of eight wavefronts shares a unit: each
// walks six rows at once, 64 consecutive entries of a row per load with the next
// 64 already requested, and looks their indices up in a bitmap of P_G instead of
// moving a cursor; four wavefronts then multiply while a fifth adds up the
// pivots' squares.  P_G is taken KC parents at a time.  Measured, the whole
// factorization in 3-D at rho = 3: 10,007 points 79.5 -> 9.5 ms, 100,000 points
// 519 -> 67 ms; bound by the walks (a window of 64 entries waits for its look-ups
// and the request behind them).
constexpr int kThreads = 512;
constexpr int kWaves = kThreads / kWave;
constexpr int kRowsPerWave = kGroupRows / kWaves;
constexpr int kTileRows = kGroupCols + kGroupRows;

typedef float mfma_f4 __attribute__((ext_vector_type(4)));

struct GroupArgs {
    const int64_t* colptr;
    const int32_t* rowidx;
    const uint32_t* csc2csr;
    const int64_t* rowptr;
    const int64_t* rowend;
    const int32_t* colidx;
    float* Lv;
    float* Lcsc;
    double* diag;
    const double* xh;
    int d;
    float ell;
    int policy;
    double tau;
    unsigned long long* counters;
    const int32_t* inst;
};

// The position of index i among the group's parents, or -1.
//  MapLookup: per 32 indices below g0 the parents' bits and the first one's
//  position, one LDS read.  SearchLookup: the parents themselves, for columns
//  whose bitmap the LDS does not hold; one read per halving.
struct MapLookup {
    struct __align__(8) Word {
        uint32_t bits, rank;
    };
    Word* map;
    __host__ __device__ static size_t bytes(int g0, int) { return (size_t(g0) / 32 + 1) * sizeof(Word); }
    __device__ __forceinline__ void build(unsigned char* lds, const int32_t* parents, int np, int g0) {
        map = reinterpret_cast<Word*>(lds);
        for (int t = threadIdx.x; t <= g0 / 32; t += kThreads) map[t] = Word{0u, 0u};
        __syncthreads();
        for (int t = threadIdx.x; t < np; t += kThreads) {
            const int i = parents[t];
            atomicOr(&map[i >> 5].bits, 1u << (i & 31));
            if (t == 0 || (parents[t - 1] >> 5) != (i >> 5)) map[i >> 5].rank = uint32_t(t);
        }
    }
    __device__ __forceinline__ int find(int i) const {  // 0 <= i < g0
        const Word w = map[i >> 5];
        const uint32_t bit = 1u << (i & 31);
        return w.bits & bit ? int(w.rank) + __popc(w.bits & (bit - 1)) : -1;
    }
};

struct SearchLookup {
    int32_t* list;
    int n;
    __host__ __device__ static size_t bytes(int, int np) { return (size_t(np) + 1) * sizeof(int32_t); }
    __device__ __forceinline__ void build(unsigned char* lds, const int32_t* parents, int np, int) {
        list = reinterpret_cast<int32_t*>(lds);
        n = np;
        for (int t = threadIdx.x; t < np; t += kThreads) list[t] = parents[t];
    }
    __device__ __forceinline__ int find(int i) const {
        int lo = 0, hi = n;  // the first position whose parent is not below i
        while (lo < hi) {
            const int mid = (lo + hi) / 2;
            if (list[mid] < i) lo = mid + 1;
            else hi = mid;
        }
        return lo < n && list[lo] == i ? lo : -1;
    }
};

template <int TWONU, int KC, typename LOOKUP>
__global__ __launch_bounds__(kThreads) void ichol_group(GroupArgs a, const kc::GroupDesc* __restrict__ groups,
                                                        const int2* __restrict__ gunits, int64_t ubeg, int64_t uend) {
    constexpr int kStride = KC + 4;  // 16 rows x 4 parents of an MFMA operand fall into 64 banks
    constexpr int kCStride = kGroupCols + 1;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float Ld[kGroupCols][kGroupCols + 1];
    __shared__ double piv[kGroupCols];
    __shared__ int pzero[kGroupCols];
    float* T = reinterpret_cast<float*>(smem);  // diagonal rows (also the second operand), then panel rows
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int64_t u = ubeg + int64_t(blockIdx.x);
    if (u >= uend) return;  // the whole workgroup
    const int2 gu = gunits[u];
    const kc::GroupDesc G = groups[gu.x];
    const int tile = gu.y;
    const int g0 = G.g0, m = G.g1 - G.g0;
    const int64_t t0 = a.rowptr[g0];
    const int np = int(a.rowend[g0] - 1 - t0);
    const int64_t cg0 = a.colptr[g0];
    // the walks of this wavefront's panel rows: row from rp, pos entries before (k, g0)
    uint32_t rp[kRowsPerWave];
    int pos[kRowsPerWave], win[kRowsPerWave];
    int idx[kRowsPerWave];
    float val[kRowsPerWave];
    {
        int k = -1, p = 0;
        uint32_t r = 0;
        const int64_t pr = int64_t(tile) * kGroupRows + wave * kRowsPerWave + lane;
        if (lane < kRowsPerWave && pr < G.nb) {
            k = a.rowidx[cg0 + m + pr];
            r = uint32_t(a.rowptr[k]);
            p = int(a.csc2csr[cg0 + m + pr] - r);
        }
#pragma unroll
        for (int q = 0; q < kRowsPerWave; ++q) {
            rp[q] = uint32_t(__builtin_amdgcn_readlane(int(r), q));
            pos[q] = __builtin_amdgcn_readlane(p, q);
            win[q] = 0;
        }
    }
    // 64 entries of row q from entry w on (rows are padded to 64 entries; past the row, its first ones)
    auto fetch = [&](int q, int w, int& i, float& v) {
        const int64_t at = int64_t(rp[q]) + (w < pos[q] ? w : 0) + lane;
        i = a.colidx[at];
        v = a.Lv[at];
    };
#pragma unroll
    for (int q = 0; q < kRowsPerWave; ++q) fetch(q, 0, idx[q], val[q]);
    LOOKUP parents;
    parents.build(smem + sizeof(float) * kTileRows * kStride, a.colidx + t0, np, g0);

    mfma_f4 acc = mfma_f4{0.f, 0.f, 0.f, 0.f};  // wavefronts 0 .. 3: 16 rows of the tile each
    double dd = 1.0;  // wavefront 4, lane g: the pivot of row g0 + g, Theta_jj = 1 less the squares, ascending
    for (int c0 = 0; c0 < np; c0 += KC) {
        const int cn = np - c0 < KC ? np - c0 : KC;
        const int last = a.colidx[t0 + c0 + cn - 1];
        for (int t = threadIdx.x; t < kGroupCols * KC; t += kThreads) {
            const int g = t / KC, q = t % KC;
            T[g * kStride + q] = g < m && q < cn ? a.Lv[a.rowptr[g0 + g] + c0 + q] : 0.f;
        }
        float4* Z = reinterpret_cast<float4*>(T + kGroupCols * kStride);
        for (int t = threadIdx.x; t < kGroupRows * kStride / 4; t += kThreads) Z[t] = float4{0.f, 0.f, 0.f, 0.f};
        __syncthreads();
        bool more = true;
        while (more) {
            more = false;
            int nidx[kRowsPerWave];
            float nval[kRowsPerWave];
#pragma unroll
            for (int q = 0; q < kRowsPerWave; ++q) fetch(q, win[q] + kWave, nidx[q], nval[q]);
#pragma unroll
            for (int q = 0; q < kRowsPerWave; ++q) {
                const bool valid = win[q] + lane < pos[q];
                const bool mine = valid && idx[q] <= last;
                const int at = parents.find(mine ? idx[q] : 0) - c0;
                if (mine && at >= 0) T[(kGroupCols + wave * kRowsPerWave + q) * kStride + at] = val[q];
                // the window is done with when none of its entries belongs to a later chunk
                if (win[q] < pos[q] && !__any(valid && idx[q] > last)) {
                    win[q] += kWave;
                    idx[q] = nidx[q];
                    val[q] = nval[q];
                    more = more || win[q] < pos[q];
                }
            }
        }
        __syncthreads();
        if (wave < 4) {
            const float* Ar = T + (wave * 16 + lane % 16) * kStride + lane / 16;
            const float* Br = T + (lane % 16) * kStride + lane / 16;
            for (int q0 = 0; q0 < cn; q0 += 64) {
                float av[16], bv[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    av[q] = Ar[q0 + 4 * q];
                    bv[q] = Br[q0 + 4 * q];
                }
#pragma unroll
                for (int q = 0; q < 16; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], bv[q], acc, 0, 0, 0);
            }
        } else if (wave == 4 && lane < kGroupCols) {
            dd = kcdev::pivot_sum(T + lane * kStride, cn, dd);  // T is zero past cn
        }
        __syncthreads();
    }
    float* C = T;  // 64 x 16
    if (wave < 4)
#pragma unroll
        for (int i = 0; i < 4; ++i) C[(wave * 16 + 4 * (lane / 16) + i) * kCStride + lane % 16] = acc[i];
    if (wave == 4 && lane < kGroupCols) piv[lane] = dd;
    __syncthreads();
    if (wave > 0) return;

    // wavefront 0 finishes: lanes 0..15 the group's diagonal rows g0 + lane, lanes 16..63 the panel rows
    int k = -1;
    int64_t eoff = -1;  // offset of (k, g0) in column g0
    if (lane < kGroupCols) {
        if (lane < m) {
            k = g0 + lane;
            eoff = lane;
        }
    } else {
        const int64_t pr = int64_t(tile) * kGroupRows + (lane - kGroupCols);
        if (pr < G.nb) {
            eoff = m + pr;
            k = a.rowidx[cg0 + eoff];
        }
    }
    const bool panel = lane >= kGroupCols && k >= 0;
    dd = lane < kGroupCols ? piv[lane] : 0.0;
    kcdev::wave_lds_sync();
    // External part: a_g = Theta_kg - C_kg.  A panel row's Theta is in Lcsc, which
    // this unit alone overwrites; the diagonal rows are recomputed by every unit of
    // the group while its first unit writes their L there, so theirs is evaluated here.
    float av[kGroupCols], Lr[kGroupCols];
    // CSC entry of (k, g0 + g): a row of the supernode by its distance from the diagonal, a row below by its place
    auto entry = [&](int g) {
        const int j = g0 + g;
        return k < G.s1 ? a.colptr[j] + (k - j) : a.colptr[j] + (G.s1 - j) + (eoff - (G.s1 - g0));
    };
#pragma unroll
    for (int g = 0; g < kGroupCols; ++g) {
        av[g] = 0.f;
        Lr[g] = 0.f;
        if (k >= 0 && g < m && (panel || lane > g)) {
            const float th = panel ? a.Lcsc[entry(g)]
                                   : kcdev::matern_f32<TWONU>(
                                         float(kcdev::dist(a.xh + int64_t(k) * a.d, a.xh + int64_t(g0 + g) * a.d, a.d)),
                                         a.ell);
            av[g] = th - C[lane * kCStride + g];
        }
    }
    // the group's columns in order: pivot from diagonal lane g, then the rows below
#pragma unroll
    for (int g = 0; g < kGroupCols; ++g) {
        if (g < m) {
            if (lane == g) {
                double pd = dd;
#pragma unroll
                for (int h = 0; h < g; ++h) pd = __builtin_fma(-double(Lr[h]), double(Lr[h]), pd);
                bool zero = false;
                if (a.policy == KC_PIVOT_ZERO) {
                    zero = !(pd > 0.0);
                } else if (!(pd > a.tau)) {
                    pd = a.tau;
                    if (tile == 0) {
                        atomicAdd(a.counters + kShifted, 1ull);
                        note_unsound(a.counters, a.inst, g0);
                    }
                }
                if (zero && tile == 0) atomicAdd(a.counters + kNonpos, 1ull);
                piv[g] = zero ? 0.0 : __builtin_sqrt(pd);
                pzero[g] = zero;
            }
            kcdev::wave_lds_sync();
            const double ljj = piv[g];
            const bool zero = pzero[g] != 0;
            if ((lane < m && lane > g) || panel) {
                float x = av[g];
#pragma unroll
                for (int h = 0; h < g; ++h) x = __builtin_fmaf(-Lr[h], Ld[g][h], x);
                Lr[g] = zero ? 0.f : float(double(x) / ljj);
                if (lane < m) Ld[lane][g] = Lr[g];
            }
            kcdev::wave_lds_sync();
        }
    }
    // write: panel rows by every unit, the diagonal block by the group's first unit
    bool bad = false;
    if (k >= 0 && (panel || tile == 0)) {
#pragma unroll
        for (int g = 0; g < kGroupCols; ++g) {
            if (g < m && (panel || lane >= g)) {
                const int64_t e = entry(g);
                const float out = lane == g ? float(piv[g]) : Lr[g];
                a.Lcsc[e] = out;
                a.Lv[a.csc2csr[e]] = out;
                if (lane == g) a.diag[g0 + g] = piv[g];
                bad = bad || !__builtin_isfinite(out);
            }
        }
    }
    const unsigned long long nf = __ballot(bad);
    if (nf && lane == 0) {
        atomicAdd(a.counters + kNonfinite, (unsigned long long)__popcll(nf));
        note_unsound(a.counters, a.inst, g0);
    }
}

// P_G by 256 parents where a level has at most a unit per CU: fewer steps of two
// barriers each (10,007 points: 9.5 ms, 10.1 ms by 128).  By 128 in larger levels:
// the tile takes 34 KB instead of 67 KB (100,000 points: 67 ms, 89 ms by 256).
// The bitmap covers all columns next to the larger tile up to some 376,000 points.
constexpr size_t kMapMost = 92 * 1024;

template <int TWONU>
hipError_t launch(const kc_factor* f, const GroupArgs& a, int64_t ub, int64_t ue, hipStream_t s) {
    auto go = [&](auto kernel, int kc, size_t lookup) {
        kernel<<<unsigned(ue - ub), kThreads, sizeof(float) * kTileRows * size_t(kc + 4) + lookup, s>>>(
            a, f->groups, f->gunits, ub, ue);
    };
    const size_t map = MapLookup::bytes(int(f->n), 0);
    if (map > kMapMost) go(ichol_group<TWONU, 128, SearchLookup>, 128, SearchLookup::bytes(0, f->max_row));
    else if (ue - ub <= f->num_cu) go(ichol_group<TWONU, 256, MapLookup>, 256, map);
    else go(ichol_group<TWONU, 128, MapLookup>, 128, map);
    return hipGetLastError();
}

}  // namespace

namespace kc {

hipError_t launch_group(const kc_factor* f, int twonu, double ell, int policy, double tau, int64_t ub, int64_t ue,
                        hipStream_t s) {
    if (ue <= ub) return hipSuccess;
    const GroupArgs a{f->colptr, f->rowidx, f->csc2csr, f->rowptr, f->rowend, f->colidx,
                      static_cast<float*>(f->L), static_cast<float*>(f->Lcsc), f->diag, f->xh, f->d, float(ell),
                      policy, tau, f->counters, f->inst};
    if (twonu == 1) return launch<1>(f, a, ub, ue, s);
    if (twonu == 3) return launch<3>(f, a, ub, ue, s);
    return launch<5>(f, a, ub, ue, s);
}

}  // namespace kc
