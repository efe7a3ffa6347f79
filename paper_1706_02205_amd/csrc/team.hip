// ICHOL(0) levels with few units: a workgroup per 64 entries of a column (gfx950).
//
// ichol_level gives every entry (k,j) one lane, which walks row k alone: a level
// lasts as long as its longest walk, a few hundred dependent steps of an LDS
// lookup and an fma each (17 us a level at 2,000 points, 72 us at 20,011 points
// in 3-D), while most of the chip is idle.  Here 16 lanes read 16 consecutive
// entries of row k at once and look their column indices up in a
// bitmap of row j's parents (a word and a value read per lane, all entries'
// lookups in flight together; a hash table measured slower, since one probe in
// some lane or other nearly always failed and each further probe cost the whole
// wavefront an LDS round trip).  What is left in sequence is the fma chain.
// Measured, a whole factorization: 2,000 points 1.71 -> 0.52 ms, 20,011 in 3-D
// 29.9 -> 5.2 ms, 50,003 on the sphere (mixed) 8.65 -> 3.6 ms, 90,601 grid points
// (mixed) 12.1 with match masks -> 6.8 ms without using them, 160,000 (FP64)
// 22.5 -> 16.7 ms.  Bound now by each level's chain of dependent loads (schedule,
// row j, row k's place, row k: 4 us with the launch) and 0.03 us per row entry.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sweep_dev.h"
#include "team.h"

using namespace kc::counter;
using namespace kcdev;

namespace {

constexpr int kWave = 64;
constexpr int kUnit = 64;   // entries of a column per unit of the schedule
// Row entries an entry's lanes take at once.  A load instruction then serves four
// entries, and the pairs of 64 entries fit in 17 KB (FP64): with 64 a workgroup
// took 67 KB and few fitted on a CU (160,000 grid points, FP64: 26.6 ms against
// 20.9 ms; 32: 25.1 ms; 8: 25.7 ms).
constexpr int kChunk = 16;
constexpr int kTeamThreads = 5 * kWave;  // four walking wavefronts and the pivot's

// One update: L_ki and L_ji, (+0, +0) where row k's entry is no parent of j.
template <typename VT>
struct __align__(2 * sizeof(VT)) Pair {
    VT a, b;
};
// Pairs of an entry's chunk, padded so that the rows of consecutive entries start
// four banks apart and the chain's 128-bit reads do not conflict.
template <typename VT>
constexpr int kPairStride = sizeof(VT) == 8 ? kChunk + 1 : kChunk + 2;

// Row j's parents as a bitmap over [0, j): per 32 indices the bits of the parents
// and the position in the row of the first of them.
struct __align__(8) MapWord {
    uint32_t bits, rank;
};
__host__ __device__ constexpr int map_words(int j) { return j / 32 + 1; }

template <typename VT>
struct TeamArgs {
    const kc::TeamUnit* units;  // of the level
    const int32_t* rowidx;
    const uint32_t* csc2csr;
    const int64_t* rowptr;
    const int32_t* colidx;
    VT* Lv;
    VT* Lcsc;
    double* diag;
    int policy;
    double tau;
    unsigned long long* counters;
    const int32_t* inst;
};

// acc <- fma(-a, b, acc) over n pairs (a multiple of 8) in ascending order, eight
// pairs read from LDS at once.  (All 16 pairs of a chunk at once took 64 registers
// in FP64 and with them a workgroup per CU: 160,000 grid points 17.9 -> 22.1 ms.)
template <typename VT>
__device__ __forceinline__ VT chain(const Pair<VT>* __restrict__ p, int n, VT acc) {
    typedef VT vec __attribute__((ext_vector_type(16 / sizeof(VT))));
    constexpr int kRead = sizeof(VT) == 8 ? 1 : 2;  // pairs per 128-bit read
    constexpr int kVec = 8 / kRead;
    const vec* s = reinterpret_cast<const vec*>(p);
    for (int t = 0; t < n; t += 8) {
        vec v[kVec];
#pragma unroll
        for (int u = 0; u < kVec; ++u) v[u] = s[t / kRead + u];
#pragma unroll
        for (int u = 0; u < kVec; ++u) {
            if constexpr (sizeof(VT) == 8) {
                acc = __builtin_fma(-v[u][0], v[u][1], acc);
            } else {
                acc = __builtin_fmaf(-v[u][0], v[u][1], acc);
                acc = __builtin_fmaf(-v[u][2], v[u][3], acc);
            }
        }
    }
    return acc;
}

// A workgroup owns ENT of the 64 entries of a unit, in column j: ENT / EPW walking
// wavefronts with EPW entries each and one more for the pivot.  Row j goes into
// LDS: its parents' values in order, and their indices as a bitmap.  A walking
// wavefront takes its entries' rows in chunks: each lane looks one index up and
// writes the pair (L_ki, L_ji) to LDS; then lanes 0 .. EPW-1 run their entries'
// chains over those pairs.  Indices that are no parents of j leave (+0, +0):
// fma(-0, +0, acc) adds -0, which leaves every acc as it is, so the updates and
// their order are those of ichol_level and L is bitwise the same.  The next
// chunk's indices and values are on their way while the chains run.
template <bool COUNT, typename VT, int EPW, int ENT>
__device__ __forceinline__ void team_unit(const TeamArgs<VT>& a, int cap, int block, unsigned char* smem) {
    constexpr int kWalkers = ENT / EPW;
    static_assert(kWalkers + 1 == kTeamThreads / kWave);
    constexpr int kParts = kUnit / ENT;  // workgroups per unit
    constexpr int kAtOnce = kWave / kChunk;  // entries whose chunks one load takes
    constexpr int kLoads = EPW / kAtOnce;
    __shared__ double piv;
    __shared__ int piv_zero;
    const kc::TeamUnit un = a.units[block / kParts];
    const int part = (block % kParts) * ENT;
    if (part >= un.count) return;  // the whole workgroup: past the column's end
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int lane = threadIdx.x % kWave;
    const int j = un.j, np = un.np, first = un.first + part;
    const int64_t t0 = un.t0;
    VT* sval = reinterpret_cast<VT*>(smem);
    Pair<VT>* pairs = reinterpret_cast<Pair<VT>*>(smem + size_t(cap) * sizeof(VT));
    MapWord* map = reinterpret_cast<MapWord*>(smem + size_t(cap) * sizeof(VT) +
                                              sizeof(Pair<VT>) * size_t(ENT) * kPairStride<VT>);

    // this wavefront's entries, one per lane: entry e = (k, j), row k from rp, pos entries before (k, j)
    const int at = part + wave * EPW + lane;
    const int64_t e = int64_t(un.e0) + at;
    const bool mine = wave < kWalkers && lane < EPW && at < un.count;
    int k = j, pos = 0;
    uint32_t rp = 0, pend = 0;
    VT acc = VT(0);
    if (mine) {
        k = a.rowidx[e];
        pend = a.csc2csr[e];
        acc = a.Lcsc[e];  // Theta_kj
        rp = uint32_t(a.rowptr[k]);
        pos = k == j ? 0 : int(pend - rp);  // the diagonal is the pivot's business
    }

    for (int s = threadIdx.x; s < map_words(j); s += blockDim.x) map[s] = MapWord{0u, 0u};
    __syncthreads();
    for (int t = threadIdx.x; t < np; t += blockDim.x) {
        const int i = a.colidx[t0 + t];
        sval[t] = a.Lv[t0 + t];
        atomicOr(&map[i >> 5].bits, 1u << (i & 31));
        if (t == 0 || (a.colidx[t0 + t - 1] >> 5) != (i >> 5)) map[i >> 5].rank = uint32_t(t);
    }
    pad_row(sval, np, int(threadIdx.x));
    __syncthreads();

    unsigned long long hits = 0;
    if (wave < kWalkers) {
        Pair<VT>* mypairs = pairs + size_t(wave) * EPW * kPairStride<VT>;
        int longest = pos;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) longest = max(longest, __shfl_xor(longest, off, kWave));
        longest = __builtin_amdgcn_readfirstlane(longest);
        // load q covers entries q * kAtOnce ..., a chunk of kChunk row entries each
        const int within = lane % kChunk;
        uint32_t rq[kLoads];
        int pq[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            rq[q] = uint32_t(__shfl(int(rp), q * kAtOnce + lane / kChunk, kWave));
            pq[q] = __shfl(pos, q * kAtOnce + lane / kChunk, kWave);
        }
        int idx[kLoads];
        VT val[kLoads];
        auto fetch = [&](int c) {
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                // whole chunks of the row (rows are padded to 64 entries); a finished row's first one
                const int64_t p = int64_t(rq[q]) + (c < pq[q] ? c : 0) + within;
                idx[q] = a.colidx[p];
                val[q] = a.Lv[p];
            }
        };
        if (longest > 0) fetch(0);
        for (int c = 0; c < longest; c += kChunk) {
            MapWord mw[kLoads];
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                if (c + within >= pq[q]) idx[q] = -1;  // not before (k, j)
                mw[q] = map[max(idx[q], 0) >> 5];
            }
            VT lji[kLoads];
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                const uint32_t bit = 1u << (idx[q] & 31);
                if (!(mw[q].bits & bit)) idx[q] = -1;
                const int at = int(mw[q].rank) + __popc(mw[q].bits & (bit - 1));
                lji[q] = sval[idx[q] >= 0 ? at : 0];
            }
#pragma unroll
            for (int q = 0; q < kLoads; ++q) {
                const bool hit = idx[q] >= 0;
                const Pair<VT> w{hit ? val[q] : VT(0), hit ? lji[q] : VT(0)};
                mypairs[(q * kAtOnce + lane / kChunk) * kPairStride<VT> + within] = w;
                if (COUNT && hit && w.b != VT(0)) ++hits;
            }
            if (c + kChunk < longest) fetch(c + kChunk);
            wave_lds_sync();
            const int n = min(kChunk, (longest - c + 7) & ~7);
            if (lane < EPW) acc = chain<VT>(mypairs + lane * kPairStride<VT>, n, acc);
            wave_lds_sync();
        }
    } else {
        double dacc = pivot_sum(sval, np, 1.0);  // from Theta_jj = 1
        bool zero = false, shift = false;
        if (a.policy == KC_PIVOT_ZERO) {
            zero = !(dacc > 0.0);
        } else if (!(dacc > a.tau)) {
            dacc = a.tau;
            shift = true;
        }
        if (lane == 0) {
            piv = zero ? 0.0 : __builtin_sqrt(dacc);
            piv_zero = zero;
            if (first == 0 && zero) atomicAdd(a.counters + kNonpos, 1ull);
            if (first == 0 && shift) {
                atomicAdd(a.counters + kShifted, 1ull);
                note_unsound(a.counters, a.inst, j);
            }
        }
        if (COUNT && first == 0)
            for (int t = lane; t < np; t += kWave) hits += sval[t] != VT(0);  // the pivot's own updates
    }
    __syncthreads();
    const double ljj = piv;
    bool bad = false;
    if (mine) {
        VT out;
        if (piv_zero) out = VT(0);
        else if (k == j) out = VT(ljj);
        else if constexpr (sizeof(VT) == 8) out = acc / ljj;
        else out = float(double(acc) / ljj);
        a.Lv[pend] = out;
        a.Lcsc[e] = out;
        if constexpr (sizeof(VT) == 4)
            if (k == j) a.diag[j] = ljj;
        bad = !__builtin_isfinite(out);
    }
    const unsigned long long nf = __ballot(bad);
    if (nf && lane == 0) {
        atomicAdd(a.counters + kNonfinite, (unsigned long long)__popcll(nf));
        note_unsound(a.counters, a.inst, j);
    }
    if (COUNT) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) hits += __shfl_xor(hits, off, kWave);
        if (lane == 0 && hits) atomicAdd(a.counters + kUpdates, hits);
    }
}

template <bool COUNT, typename VT, int EPW, int ENT>
__global__ __launch_bounds__(kTeamThreads) void ichol_team(TeamArgs<VT> a, int cap) {
    extern __shared__ __align__(16) unsigned char smem[];
    team_unit<COUNT, VT, EPW, ENT>(a, cap, blockIdx.x, smem);
}

// A level of the factorization and, in the workgroups from nteam on, a level of
// the forward sweep: rows [rbeg, rend), `passes` times over for more than 8
// right-hand sides.  The sweep's level is an earlier one than the factorization's,
// so neither reads what the other writes.
template <typename VT, int EPW, int ENT, int NR>
__global__ __launch_bounds__(kTeamThreads) void ichol_team_fwd(TeamArgs<VT> a, int cap, int nteam, SweepArgs<VT> sw, int nrhs, int64_t rbeg, int rows) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (int(blockIdx.x) < nteam) {
        team_unit<false, VT, EPW, ENT>(a, cap, blockIdx.x, smem);
        return;
    }
    const int block = int(blockIdx.x) - nteam;
    sw.r0 = block / rows * kMaxRhs;
    sweep_row<VT, NR, kTeamThreads, true>(sw, sw.rows[rbeg + block % rows], min(kMaxRhs, nrhs - sw.r0),
                                          reinterpret_cast<double*>(smem));
}

int32_t team_cap(int32_t max_row) { return (max_row + 16) / 16 * 16; }

template <int V>
using Int = std::integral_constant<int, V>;

template <typename VT>
TeamArgs<VT> team_args(const kc_factor* f, int level, int policy, double tau) {
    return {f->team_units + f->team_off[size_t(level)], f->rowidx, f->csc2csr, f->rowptr, f->colidx,
            static_cast<VT*>(f->L), static_cast<VT*>(f->Lcsc), f->diag, policy, tau,
            f->counters, f->inst};
}

// The split of a level.  At most a quarter of a unit per CU: 16 entries to a
// workgroup, 4 to a wavefront, so that the chains' LDS reads (a whole instruction
// for a wavefront's few entries) spread over more CUs.  Up to 2 units per CU: 32
// and 8, in five wavefronts as everywhere: whole units of 64 and 8, in nine, ran one
// to a CU, and a level of 257 units took twice as long as one of 256 (2,000 points 0.565 -> 0.516 ms, 20,011
// in 3-D 5.35 -> 5.19 ms with both).  Beyond, 64 and 16: half as many chain reads
// per update (160,000 grid points: 17.9 ms against 20.3 ms with 8 entries to a
// wavefront; 32: 19.5 ms).
template <typename Fn>
void team_shape(const kc_factor* f, int64_t units, Fn fn) {
    const int64_t cus = std::max(1, f->num_cu);
    if (4 * units <= cus) fn(Int<4>(), Int<16>());
    else if (units <= 2 * cus) fn(Int<8>(), Int<32>());
    else fn(Int<16>(), Int<64>());
}

}  // namespace

namespace kc {

size_t team_lds(int32_t max_row, int32_t max_col, size_t vt) {
    const size_t pair_row = vt == 8 ? kPairStride<double> : kPairStride<float>;
    return size_t(team_cap(max_row)) * vt + size_t(kUnit) * pair_row * 2 * vt +
           size_t(map_words(max_col)) * sizeof(MapWord);
}

template <typename VT>
hipError_t launch_team(const kc_factor* f, bool count, int policy, double tau, int level, hipStream_t s) {
    const int64_t units = f->team_off[size_t(level) + 1] - f->team_off[size_t(level)];
    if (units <= 0) return hipSuccess;
    const TeamArgs<VT> a = team_args<VT>(f, level, policy, tau);
    const size_t lds = team_lds(f->max_row, f->level_last[size_t(level)], sizeof(VT));
    const int32_t cap = team_cap(f->max_row);
    team_shape(f, units, [&](auto epw, auto ent) {
        constexpr int EPW = decltype(epw)::value, ENT = decltype(ent)::value;
        const unsigned grid = unsigned(units) * (kUnit / ENT);
        if (count) ichol_team<true, VT, EPW, ENT><<<grid, kTeamThreads, lds, s>>>(a, cap);
        else ichol_team<false, VT, EPW, ENT><<<grid, kTeamThreads, lds, s>>>(a, cap);
    });
    return hipGetLastError();
}

template <typename VT>
hipError_t launch_team_fwd(const kc_factor* f, int policy, double tau, int level, const double* b, double* y, int nrhs,
                           int64_t rb, int64_t re, hipStream_t s) {
    const int nl = int(f->team_off.size()) - 1;
    const int64_t rows = re - rb;
    const int64_t units = level < nl ? f->team_off[size_t(level) + 1] - f->team_off[size_t(level)] : 0;
    if (units <= 0 && rows <= 0) return hipSuccess;
    const TeamArgs<VT> a = team_args<VT>(f, level, policy, tau);
    const SweepArgs<VT> sw = fwd_args<VT>(f, b, nrhs, 0, y);
    const int32_t cap = team_cap(f->max_row);
    const int64_t passes = (nrhs + kMaxRhs - 1) / kMaxRhs;
    team_shape(f, units, [&](auto epw, auto ent) {
        constexpr int EPW = decltype(epw)::value, ENT = decltype(ent)::value;
        const int nteam = int(units) * (kUnit / ENT);
        auto go = [&](auto w) {
            constexpr int NR = decltype(w)::value;
            size_t lds = units > 0 ? team_lds(f->max_row, f->level_last[size_t(level)], sizeof(VT)) : 0;
            if (rows > 0) lds = std::max(lds, sweep_lds(NR, kTeamThreads) * sizeof(double));
            ichol_team_fwd<VT, EPW, ENT, NR><<<unsigned(nteam) + unsigned(rows * passes), kTeamThreads, lds, s>>>(
                a, cap, nteam, sw, nrhs, rb, int(std::max<int64_t>(rows, 1)));
        };
        if (nrhs == 1) go(Int<1>());
        else if (nrhs == 2) go(Int<2>());
        else if (nrhs <= 4) go(Int<4>());
        else go(Int<8>());
    });
    return hipGetLastError();
}

template hipError_t launch_team_fwd<double>(const kc_factor*, int, double, int, const double*, double*, int, int64_t,
                                             int64_t, hipStream_t);
template hipError_t launch_team_fwd<float>(const kc_factor*, int, double, int, const double*, double*, int, int64_t,
                                             int64_t, hipStream_t);
template hipError_t launch_team<double>(const kc_factor*, bool, int, double, int, hipStream_t);
template hipError_t launch_team<float>(const kc_factor*, bool, int, double, int, hipStream_t);

}  // namespace kc
