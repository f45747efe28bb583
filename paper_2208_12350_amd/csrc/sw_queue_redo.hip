// sw_queue_redo.hip -- second look at the pairs whose reverse sweep found no
// start (the redo list, see sw_sweep.h): a drifted forward sweep gives the
// exact score and end row of a pair, but on rare ties an end column that is
// too small.
//
// For each listed pair the kernel finds the end column (the first column of
// the end row that holds the score), then the start as the reverse sweep
// does.  Both are the same search for the row-major-first cell that holds a
// known score, with scores read from the byte tables, so one kernel serves
// every scheme: two pairs per wavefront (64-lane groups) up to 512 rows, per
// workgroup (the cooperative sweep) above.  Few pairs are listed, so what
// counts is the time of one: the forward search sweeps only the columns and
// rows an alignment that ends past the column found can use, and in a
// wavefront ends at the first hit.  A pair of 2000 x 6000 took 7.6 ms in one
// wavefront, at the end of 1,000,000 mixed pairs, and takes 3.3 in
// four.  A launch without listed pairs costs its workgroups one load.
#include "sw_coop.h"
#include "sw_queue.h"

namespace sw {

namespace {

// Row-major-first cell of each of two jobs (packed int16, pair A low) that
// holds the job's score (J.fwd_score, 0 = no job); row kNoRow if there is
// none.  With `first_hit` the search of both ends as soon as each has a cell.
// The result is the same in every lane.
template <int R>
__device__ __forceinline__ void find_score(const KParams& P, const SchemeLds& S, uint16_t* wbuf, const PairJob& JA,
                                           const PairJob& JB, bool first_hit, int lane, int (&row)[2], int (&col)[2]) {
    constexpr int W = 64;
    using Stager = RefStager<W>;
    constexpr uint32_t K = kI16Bias;
    constexpr uint32_t K2 = K | (K << 16);
    const int l = lane;
    const int mmax = imax(JA.m, JB.m);
    const int steps = __builtin_amdgcn_readfirstlane(mmax > 0 ? mmax + W - 1 : 0);
    uint16_t* bufA = wbuf;
    uint16_t* bufB = wbuf + Stager::kBuf;
    Stager stA, stB;
    stA.load(P.refs, JA, P.order, 0, l);
    stB.load(P.refs, JB, P.order, 0, l);
    const int AA = S.alphabet[JA.sid], AB = S.alphabet[JB.sid];
    uint32_t apk[R];
    {
        int rawA[R], rawB[R];
        const int remA = load_rows<R>(P, JA, l, rawA), remB = load_rows<R>(P, JB, l, rawB);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t a = (r < remA) & (rawA[r] < AA) ? rawA[r] : kPad;
            const uint32_t b = (r < remB) & (rawB[r] < AB) ? rawB[r] : kPad;
            apk[r] = a | (b << 16);
        }
    }
    int bad = -1;   // residues were checked by the first sweeps
    stA.store(bufA, JA, AA, 0, l, bad);
    stB.store(bufB, JB, AB, 0, l, bad);
    const u16x2 go2 = pk(cost16(S.gap_open[JA.sid]) | (cost16(S.gap_open[JB.sid]) << 16));
    const u16x2 ge2 = pk(cost16(S.gap_extend[JA.sid]) | (cost16(S.gap_extend[JB.sid]) << 16));
    const u16x2 zero = pk(K2);
    // one below the biased score; out of reach for no job
    const uint32_t tA = JA.fwd_score > 0 ? K + (uint32_t)JA.fwd_score - 1u : 0x7C00u;
    const uint32_t tB = JB.fwd_score > 0 ? K + (uint32_t)JB.fwd_score - 1u : 0x7C00u;
    const u16x2 thr = pk(tA | (tB << 16));
    wave_lds_sync();

    u16x2 H[R], E[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { H[r] = zero; E[r] = zero; }
    uint32_t Hlast = K2, Flast = K2, Hup_prev = K2;
    const uint16_t* rblA = bufA + W - l;
    const uint16_t* rblB = bufB + W - l;
    u16x2 sc[R];
    int bbA_next = 0, bbB_next = 0;
    int rA = kNoRow, rB = kNoRow, cA = 0, cB = 0;
    bool stop = false;
    for (int t0 = 0; t0 < steps && !stop; t0 += kChunk) {
        if (t0 > 0) {
            wave_lds_sync();
            stA.store(bufA, JA, AA, t0, l, bad);
            stB.store(bufB, JB, AB, t0, l, bad);
            wave_lds_sync();
        }
        if (t0 + kChunk < steps) {
            stA.load(P.refs, JA, P.order, t0 + kChunk, l);
            stB.load(P.refs, JB, P.order, t0 + kChunk, l);
        }
        const int a0 = rblA[0], b0 = rblB[0];
#pragma unroll
        for (int r = 0; r < R; ++r) sc[r] = load_scores(S.mat, a0 + (int)(apk[r] & 0xFFFF), b0 + (int)(apk[r] >> 16));
        bbA_next = rblA[1];
        bbB_next = rblB[1];
        const int tn = __builtin_amdgcn_readfirstlane(steps - t0 < kChunk ? steps - t0 : kChunk);
        for (int tt = 0; tt < tn && !stop; ++tt) {
            const int bbA2 = rblA[tt + 2];
            const int bbB2 = rblB[tt + 2];
            const u16x2 Hup = pk((uint32_t)shift_in_group<W>((int)Hlast, (int)K2));
            u16x2 F = pk((uint32_t)shift_in_group_zero<W>((int)Flast));
            u16x2 diag = pk(Hup_prev);
            Hup_prev = u32(Hup);
            u16x2 Hmu = pk_sat_sub(Hup, go2);
            u16x2 top = zero;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                F = pk_max3(pk_sat_sub(F, ge2), Hmu, zero);
                const u16x2 h = pk_max3(diag + sc[r], E[r], F);
                sc[r] = load_scores(S.mat, bbA_next + (int)(apk[r] & 0xFFFF), bbB_next + (int)(apk[r] >> 16));
                diag = H[r];
                H[r] = h;
                Hmu = pk_sat_sub(h, go2);
                E[r] = pk_max3(pk_sat_sub(E[r], ge2), Hmu, zero);
                top = pk_max(top, h);
            }
            Hlast = u32(H[R - 1]);
            Flast = u32(F);
            bbA_next = bbA2;
            bbB_next = bbB2;
            if (__builtin_amdgcn_ballot_w64(u32(pk_sat_sub(top, thr)) != 0) != 0) {
                int hitA = kNoRow, hitB = kNoRow;
#pragma unroll
                for (int r = R - 1; r >= 0; --r) {
                    const uint32_t w = u32(pk_sat_sub(H[r], thr));
                    hitA = (w & 0xFFFFu) ? l * R + r : hitA;
                    hitB = (w >> 16) ? l * R + r : hitB;
                }
                const int j = t0 + tt - l;
                cA = hitA < rA ? j : cA;
                cB = hitB < rB ? j : cB;
                rA = hitA < rA ? hitA : rA;
                rB = hitB < rB ? hitB : rB;
                if (first_hit)
                    stop = (JA.fwd_score <= 0 || __builtin_amdgcn_ballot_w64(rA != kNoRow) != 0) &&
                           (JB.fwd_score <= 0 || __builtin_amdgcn_ballot_w64(rB != kNoRow) != 0);
            }
        }
    }
    row[0] = rA; row[1] = rB;
    col[0] = cA; col[1] = cB;
#pragma unroll
    for (int p = 0; p < 2; ++p)
        for (int off = 1; off < W; off <<= 1) {
            const int oi = __shfl_xor(row[p], off);
            const int oj = __shfl_xor(col[p], off);
            col[p] = oi < row[p] ? oj : col[p];
            row[p] = oi < row[p] ? oi : row[p];
        }
    wave_lds_sync();   // the next search rewrites the reference buffers
}

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

// Whether the pair holds a residue outside its scheme's alphabet (a call that
// does not check them, option validate = 0).  The sweeps and the searches
// here score such a residue differently, so a search may then fail.
__device__ __forceinline__ bool has_invalid(const KParams& P, const Listed& x) {
    const int A = P.alphabet[x.sid], lane = (int)__lane_id();
    const int n = (int)(P.q_end[x.pair] - x.q0);
    bool bad = false;
    for (int i = lane; i < n; i += 64) bad |= P.queries[x.q0 + i] >= A;
    for (int j = lane; j < x.m0; j += 64) bad |= P.refs[x.r0 + j] >= A;
    return __builtin_amdgcn_ballot_w64(bad) != 0;
}

// Redo of two pairs.  search(J, first_hit, row, col) finds the cells of their
// jobs; max_rows is the most rows it can take, and the thread with `writes`
// set writes.
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
        search(J, round == 0, row, col);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (x[p].pair < 0) continue;
            // the end row is exact, so a hit elsewhere is an error too
            if (row[p] == kNoRow || (round == 0 && row[p] != J[p].n - 1)) {
                if (P.validate || !has_invalid(P, x[p])) {
                    atomicOr(&P.flags[kFlagReverseMismatch], 1);
                } else if (writes) {
                    // no result is defined for the pair: it starts where it ends
                    sw_result* o = P.out + x[p].pair;
                    o->q_start = x[p].qe;
                    o->r_start = o->r_end = x[p].re;
                }
                x[p].pair = -1;
                continue;
            }
            if (round == 0) {
                x[p].re = J[p].fwd_re + col[p];
                continue;
            }
            if (writes) {
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

// The entries k and k + 1 of the list, and their rows (the larger).
__device__ __forceinline__ int listed_rows(const KParams& P, int k, int n, int n_pairs, int (&id)[2]) {
    int rows = 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        id[p] = k + p < n ? __builtin_amdgcn_readfirstlane(P.redo[k + p]) : -1;
        if (id[p] >= n_pairs) {
            atomicOr(&P.flags[kFlagInternal], 1);
            id[p] = -1;
        }
        if (id[p] >= 0) rows = imax(rows, (int)(P.q_end[id[p]] - P.q_beg[id[p]]));
    }
    return __builtin_amdgcn_readfirstlane(rows);
}

template <int R>
__device__ __forceinline__ void redo_wave(const KParams& P, const SchemeLds& S, uint16_t* wbuf, const int (&id)[2],
                                          int lane, const int8_t* lut, const BinInfo* bins,
                                          unsigned long long* counters) {
    redo_pairs(P, id[0], id[1], 64 * R, lane == 0, lut, bins, counters,
               [&](const PairJob (&J)[2], bool first_hit, int (&row)[2], int (&col)[2]) {
                   find_score<R>(P, S, wbuf, J[0], J[1], first_hit, lane, row, col);
               });
}

template <int R>
__device__ __forceinline__ void redo_coop(const KParams& P, const SchemeLds& S, CoopLds& C, const int (&id)[2],
                                          int tid, const int8_t* lut, const BinInfo* bins,
                                          unsigned long long* counters) {
    redo_pairs(P, id[0], id[1], kCoopW * R, tid == 0, lut, bins, counters,
               [&](const PairJob (&J)[2], bool, int (&row)[2], int (&col)[2]) {
                   int best[2];
                   __syncthreads();   // the last search's LDS is free
                   coop_best<R>(P, S, C, J[0], J[1], tid, best, row, col);
#pragma unroll
                   for (int p = 0; p < 2; ++p)
                       if (best[p] != J[p].fwd_score || best[p] == 0) row[p] = kNoRow;
               });
}

// (one wavefront per SIMD: few are in flight)
constexpr int kRedoTall = 512;   // rows above which a workgroup searches together
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, 1))) void sw_redo_kernel(
    KParams P, const int8_t* lut, const BinInfo* bins, unsigned long long* counters) {
    __shared__ __attribute__((aligned(16))) SchemeLds L;
    __shared__ uint16_t wbufs[kWavesPerBlock * 2 * RefStager<64>::kBuf];
    __shared__ CoopLds C;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_pairs = __builtin_amdgcn_readfirstlane(*P.n_dev);
    int n = __builtin_amdgcn_readfirstlane(__atomic_load_n(&P.meta[kMetaRedo], __ATOMIC_RELAXED));
    n = n < n_pairs ? n : n_pairs;
    if (2 * (int)blockIdx.x >= n) return;
    if (blockIdx.x == 0 && tid == 0) counters[kCtrRedoPairs] = (unsigned long long)n;
    load_schemes(L, P, tid);
    __syncthreads();
    uint16_t* wbuf = wbufs + wave * 2 * RefStager<64>::kBuf;
    int id[2];
    // the tall pairs first: the same entries in every wavefront, so every
    // barrier is reached by the whole workgroup
    for (int k = 2 * (int)blockIdx.x; k < n; k += 2 * (int)gridDim.x) {
        const int rows = listed_rows(P, k, n, n_pairs, id);
        if (rows <= kRedoTall) continue;
        if (rows <= 768) redo_coop<3>(P, L, C, id, tid, lut, bins, counters);
        else if (rows <= 1024) redo_coop<4>(P, L, C, id, tid, lut, bins, counters);
        else if (rows <= 1536) redo_coop<6>(P, L, C, id, tid, lut, bins, counters);
        else redo_coop<8>(P, L, C, id, tid, lut, bins, counters);
    }
    for (int k = 2 * ((int)blockIdx.x + (int)gridDim.x * wave); k < n; k += 2 * kWavesPerBlock * (int)gridDim.x) {
        const int rows = listed_rows(P, k, n, n_pairs, id);
        if (rows > kRedoTall) continue;
        if (rows <= 256) redo_wave<4>(P, L, wbuf, id, lane, lut, bins, counters);
        else redo_wave<8>(P, L, wbuf, id, lane, lut, bins, counters);
    }
}

}  // namespace

hipError_t launch_redo(const KParams& P, const int8_t* lut, const BinInfo* bins, unsigned long long* counters,
                       int blocks, hipStream_t s) {
    hipLaunchKernelGGL(sw_redo_kernel, dim3(blocks > 0 ? blocks : 1), dim3(kBlock), 0, s, P, lut, bins, counters);
    return hipGetLastError();
}

}  // namespace sw
