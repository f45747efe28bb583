// sw_queue_redo.hip -- second look at the pairs whose reverse sweep found no
// start (the redo list, see sw_sweep.h): a drifted forward sweep gives the
// exact score and end row of a pair, but on rare ties an end column that is
// too small.
//
// For each listed pair the kernel finds the end column (the first column of
// the end row that holds the score), then the start.  Both are the search of
// the reverse sweep for the row-major-first cell that holds a known score, and
// are made by it, forwards for the end, with the pair's own score source:
// two pairs per wavefront (64-lane groups) up to 512 rows, per cooperative
// group above.  The search for the end sweeps only the columns and rows an
// alignment that ends past the column found can use.  With byte tables and a
// barrier in every step above 512 rows, 3,000 low-complexity DNA pairs of 1000 to
// 2000 residues at a match of 10, 45 of them listed, took 7.4 ms, now 5.5 (7.2
// with no drift and no list); 20,000 pairs of 600 to 1000 built so that 14,000 are
// listed 25.0, now 11.1 (8.7).  A launch without listed pairs costs its
// workgroups one load.
#include "sw_coop.h"
#include "sw_queue.h"

namespace sw {

namespace {

__device__ __forceinline__ PairJob no_job() {
    PairJob J;
    J.dir = 1; J.n = 0; J.m = 0; J.qbase = 0; J.rbase = 0; J.sid = 0;
    J.fwd_score = 0; J.fwd_qe = -1; J.fwd_re = -1;
    return J;
}

// One listed pair: its span, result so far and scheme.
struct Listed {
    int pair, sid, S, qe, re, m0;
    int64_t q0, r0;
};

__device__ __forceinline__ Listed listed(const KParams& P, int pair) {
    Listed x;
    x.pair = -1; x.sid = 0; x.S = 0; x.qe = x.re = -1; x.m0 = 0; x.q0 = x.r0 = 0;
    if (pair < 0) return x;
    const sw_result r = P.out[pair];
    const int64_t n0 = P.q_end[pair] - P.q_beg[pair], m0 = P.r_end[pair] - P.r_beg[pair];
    const int sid = P.scheme_id ? (int)P.scheme_id[pair] : 0;
    if (r.score <= 0 || r.q_end < 0 || r.q_end >= n0 || n0 > SW_MAX_QUERY || r.r_end < 0 || r.r_end >= m0 ||
        m0 > kI16MaxRef || sid >= SW_MAX_SCHEMES) {
        atomicOr(&P.flags[kFlagInternal], 1);
        return x;
    }
    x.pair = pair; x.sid = sid; x.S = r.score; x.qe = r.q_end; x.re = r.r_end; x.m0 = (int)m0;
    x.q0 = P.q_beg[pair];
    x.r0 = P.r_beg[pair];
    return x;
}

// Search for the end column: the part of the pair that an alignment of
// score S that ends in row qe, past column re, can use.
__device__ __forceinline__ PairJob end_job(const KParams& P, const Listed& x) {
    PairJob J = no_job();
    if (x.pair < 0) return J;
    int n = x.qe + 1, m = x.m0;
    reverse_extent(x.S, P.max_score[x.sid], P.gap_open[x.sid], P.gap_extend[x.sid], n, m);
    const int c0 = imax(0, x.re + 2 - m);
    J.sid = x.sid;
    J.n = n;
    J.m = x.m0 - c0;
    J.qbase = x.q0 + x.qe + 1 - n;
    J.rbase = x.r0 + c0;
    J.fwd_score = x.S;
    J.fwd_re = c0;   // column of the job's first
    return J;
}

__device__ __forceinline__ PairJob start_job(const KParams& P, const Listed& x) {
    PairJob J = no_job();
    if (x.pair < 0) return J;
    J.sid = x.sid;
    J.n = x.qe + 1;
    J.m = x.re + 1;
    J.dir = -1;
    J.qbase = x.q0 + x.qe;
    J.rbase = x.r0 + x.re;
    J.fwd_score = x.S;
    reverse_extent(x.S, P.max_score[x.sid], P.gap_open[x.sid], P.gap_extend[x.sid], J.n, J.m);
    return J;
}

// Redo of two pairs.  search(J, row, col) finds the cells of their jobs;
// max_rows is the most rows it can take, and the first lane of the wavefront
// with `writes` set writes.
template <class Search>
__device__ __forceinline__ void redo_pairs(const KParams& P, int pairA, int pairB, int max_rows, bool writes,
                                           const int8_t* lut, const BinInfo* bins, unsigned long long* counters,
                                           Search&& search) {
    Listed x[2] = {listed(P, pairA), listed(P, pairB)};
    long long was[2] = {0, 0};
    int bin[2] = {-1, -1};
#pragma unroll 1
    for (int round = 0; round < 2; ++round) {
        PairJob J[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            J[p] = round == 0 ? end_job(P, x[p]) : start_job(P, x[p]);
            if (J[p].n > max_rows) {   // cannot happen: R was chosen for the pair's rows
                atomicOr(&P.flags[kFlagInternal], 1);
                J[p] = no_job();
                x[p].pair = -1;
            }
            if (round == 0 && x[p].pair >= 0) {
                const PairJob old = start_job(P, x[p]);   // what the statistics counted
                was[p] = (long long)old.n * old.m;
                bin[p] = lut[(P.col_ok[x[p].sid] ? kLutI16Col : kLutI16) * kLutRows + (old.n - 1) / 16];
            }
        }
        int row[2], col[2];
        search(J, row, col);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (x[p].pair < 0) continue;
            // the end row is exact, so a hit elsewhere is an error too
            if (row[p] == kNoRow || (round == 0 && row[p] != J[p].n - 1)) {
                atomicOr(&P.flags[kFlagReverseMismatch], 1);
                x[p].pair = -1;
                continue;
            }
            if (round == 0) {
                x[p].re = J[p].fwd_re + col[p];
                continue;
            }
            if (writes && item_lane() == 0) {
                sw_result* o = P.out + x[p].pair;
                o->q_start = x[p].qe - row[p];
                o->r_start = x[p].re - col[p];
                o->r_end = x[p].re;
                // the reverse cells, counted at planning for the old end
                const unsigned long long more = (unsigned long long)((long long)J[p].n * J[p].m - was[p]);
                if (more && bin[p] >= 0 && bin[p] < kMaxBins) {
                    atomicAdd(&counters[kCtrRevCells], more);
                    atomicAdd(&counters[kCtrBinCells + kMaxBins + bin[p]], more);
                    if (P.col_ok[x[p].sid] && bins[bin[p]].col)
                        atomicAdd(&counters[kCtrBinColCells + kMaxBins + bin[p]], more);
                }
            }
        }
    }
}

// The entries k and k + 1 of the list that score source VAR (and the launch's
// drift group) serves, -1 for others, and their rows (the larger).
template <int VAR>
__device__ __forceinline__ int listed_rows(const KParams& P, int k, int n, int n_pairs, int (&id)[2]) {
    int rows = 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        id[p] = k + p < n ? __builtin_amdgcn_readfirstlane(P.redo[k + p]) : -1;
        if (id[p] >= n_pairs) {
            atomicOr(&P.flags[kFlagInternal], 1);
            id[p] = -1;
        }
        if (id[p] < 0) continue;
        const int sid = P.scheme_id ? (int)P.scheme_id[id[p]] & (SW_MAX_SCHEMES - 1) : 0;
        const bool own = VAR == kVarCol ? P.col_ok[sid] && drift_group(P, sid) == P.group : sid == P.ptab_sid;
        if (!__builtin_amdgcn_readfirstlane((int)own)) id[p] = -1;
        else rows = imax(rows, (int)(P.q_end[id[p]] - P.q_beg[id[p]]));
    }
    return __builtin_amdgcn_readfirstlane(rows);
}

template <int VAR, int R, bool COOP>
__device__ __forceinline__ void redo(const KParams& P, CoopWork<VAR, 8>& K, int idA, int idB, int tid, int wave,
                                     const int8_t* lut, const BinInfo* bins, unsigned long long* counters) {
    using Src = typename std::conditional<VAR == kVarPtab, PtabScores<64, R, kChunk>, ColScores<64, R, kChunk>>::type;
    redo_pairs(P, idA, idB, (COOP ? kCoopW : 64) * R, !COOP || wave == 0, lut, bins, counters,
               [&](const PairJob (&J)[2], int (&row)[2], int (&col)[2]) {
        if (COOP) __syncthreads();   // the last search's LDS is free
        else wave_lds_sync();
        sweep_jobs<Src, 64, R, true, kChunk, COOP>(
            P, K.L, reinterpret_cast<uint16_t*>(K.wbufs[wave]), J[0], J[1], J[0].fwd_score > 0 ? idA : -1,
            J[1].fwd_score > 0 ? idB : -1, item_lane(), &K.X, wave,
            [&](const int (&r)[2], const int (&c)[2]) {
                row[0] = r[0]; row[1] = r[1];
                col[0] = c[0]; col[1] = c[1];
            });
    });
}

constexpr int kRedoTall = 512;   // rows above which a workgroup searches together

// The listed pairs of one score source.
template <int VAR>
__device__ __forceinline__ void redo_source(const KParams& P, CoopWork<VAR, 8>& K, int n, int n_pairs, int tid, int wave,
                                            const int8_t* lut, const BinInfo* bins, unsigned long long* counters) {
    __syncthreads();
    K.load(P, tid);
    __syncthreads();
    int id[2];
    // the tall pairs first: the same entries in every wavefront, so every
    // barrier is reached by the whole workgroup
    for (int k = 2 * (int)blockIdx.x; k < n; k += 2 * (int)gridDim.x) {
        const int rows = listed_rows<VAR>(P, k, n, n_pairs, id);
        if (rows <= kRedoTall) continue;
        if (rows <= 1024) redo<VAR, 4, true>(P, K, id[0], id[1], tid, wave, lut, bins, counters);
        else redo<VAR, 8, true>(P, K, id[0], id[1], tid, wave, lut, bins, counters);
    }
    for (int k = 2 * ((int)blockIdx.x + (int)gridDim.x * wave); k < n; k += 2 * kWavesPerBlock * (int)gridDim.x) {
        const int rows = listed_rows<VAR>(P, k, n, n_pairs, id);
        if (rows > kRedoTall || rows == 0) continue;
        if (rows <= 256) redo<VAR, 4, false>(P, K, id[0], id[1], tid, wave, lut, bins, counters);
        else redo<VAR, 8, false>(P, K, id[0], id[1], tid, wave, lut, bins, counters);
    }
}

__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) void sw_redo_kernel(
    KParams P, const int8_t* lut, const BinInfo* bins, unsigned long long* counters) {
    using Col = CoopWork<kVarCol, 8>;
    using Ptab = CoopWork<kVarPtab, 8>;
    __shared__ __attribute__((aligned(16))) char lds[sizeof(Col) > sizeof(Ptab) ? sizeof(Col) : sizeof(Ptab)];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_pairs = __builtin_amdgcn_readfirstlane(*P.n_dev);
    int n = __builtin_amdgcn_readfirstlane(__atomic_load_n(&P.meta[kMetaRedo], __ATOMIC_RELAXED));
    n = n < n_pairs ? n : n_pairs;
    if (2 * (int)blockIdx.x >= n) return;
    if (blockIdx.x == 0 && tid == 0) counters[kCtrRedoPairs] = (unsigned long long)n;
    if (P.n_drift > 0) redo_source<kVarCol>(P, *reinterpret_cast<Col*>(lds), n, n_pairs, tid, wave, lut, bins, counters);
    if (P.ptab_sid >= 0 && P.group == 0) redo_source<kVarPtab>(P, *reinterpret_cast<Ptab*>(lds), n, n_pairs, tid, wave, lut, bins, counters);
}

}  // namespace

hipError_t launch_redo(const KParams& P, const int8_t* lut, const BinInfo* bins, unsigned long long* counters,
                       int blocks, hipStream_t s) {
    hipLaunchKernelGGL(sw_redo_kernel, dim3(blocks > 0 ? blocks : 1), dim3(kBlock), 0, s, P, lut, bins, counters);
    return hipGetLastError();
}

}  // namespace sw
