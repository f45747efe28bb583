// sw_sweep.h -- the forward/reverse sweep of one wavefront work item (gfx950).
//
// Hot path: the forward and reverse sweeps of the affine-gap Smith-Waterman
// (Gotoh) recurrences of Section II-B-1 / Fig. 2, batched over many
// independent query/reference pairs.
//
// Mapping onto CDNA4 (one pair per lane group, anti-diagonal sweep):
//   * A wavefront (64 lanes) is split into 64/W groups of W lanes (W = 16,
//     32 or 64).  Each group owns one pair.  Lane l of a group owns query rows
//     l*R .. l*R+R-1 in registers (H, E and the row's running best), so a
//     group covers W*R >= n rows in a single sweep.
//   * At step t lane l computes column j = t - l for its R rows, i.e. the
//     group sweeps anti-diagonals of lane-blocks.  The value a lane needs from
//     the row above its block (H and F of the last row of lane l-1 at
//     column j) was produced by lane l-1 one step earlier and arrives through
//     a DPP row/wave shift -- the same mechanism for every lane, with no
//     divergent first-lane path (the lesson of Section VI-A).  Lane 0 of a
//     group receives zeros, the matrix's top boundary.
//   * The reference of each group is staged in LDS as pre-scaled row offsets
//     into the LDS substitution matrix, so one LDS byte read per cell gives
//     M[a_i][b_j].  Columns left of 0 (ramp-up) and right of m (ramp-down)
//     read a padding code whose score is -1.
//   * No per-step barrier or warp vote: a wavefront runs in lock-step
//     (Section VI-B), and shared state is initialised once, by the lanes that
//     use it (Section VI-C).
//
// Exactness of the padding: E and F are carried clamped at zero
// (E* = max(E, 0)), which leaves H unchanged because H takes a max with 0.  A
// padded cell (row >= n or column >= m or < 0) scores at most
// max(diag - 1, E, F) where diag <= S and E, F <= S - o, so with o >= 1 it is
// strictly below the pair's best S and never changes S or its first cell;
// real cells never depend on padded ones (they lie below or to the right).
//
// Packed int16 variant (sweep_i16):
// Same anti-diagonal lane-group sweep as the int32 kernel, but every 32-bit
// register carries two independent pairs: pair A in the low 16 bits and pair
// B in the high 16 bits, so one packed VALU instruction (v_pk_*_i16/u16)
// advances two cells.  A W-lane group therefore aligns two pairs, and the
// host pairs them up from the same length bin (similar query and reference
// lengths, so little padding).
//
// Biased values: every H, E and F of the packed path is stored plus a bias
// K = kI16Bias (1024), so "zero" is K.  All stored values then lie in
// [K, 0x7BFF]: bit patterns of positive normal half-precision numbers, whose
// numeric order is their integer order.  A three-way maximum of two packed
// halves is therefore one v_pk_maximum3_f16 on the raw patterns (it never
// rounds: it returns one of its inputs).  The clamps E* = max(E, 0) and
// F* = max(F, 0) become a third operand K of that maximum, and with E, F >= K
// the clamp of H at zero comes for free: H = max3(diag + M[a][b], E, F).
// diag + M[a][b] may fall below K (a mismatch next to a zero cell), even
// into the denormal range, but it is then below E >= K and never selected.
//
// Range: the host routes a pair here only when min(n, m) * max_score <=
// kI16Limit, which keeps K + H + max_score <= 0x7BFF for every cell of the
// pair (and of its reverse sweep, whose values never exceed the forward
// maximum), and when m <= kI16MaxRef, which keeps the column field of the
// keys below to 15 bits.
//
// Row best: rows r (even) and r+1 of a lane share one 32-bit key per pair,
// (H << 16) | (rowbit << 15) | (kColMax - j) with rowbit = 1 for row r.  An
// unsigned max (v_max3_u32 over both rows) keeps the largest H, then the
// upper row, then the smallest column j: the row-major-first maximum of the
// two rows.
#pragma once

#include <type_traits>

#include "sw_device.h"
#include "sw_internal.h"

namespace sw {

// LDS reference buffer of one wavefront (in 16-bit entries), sized for the
// widest layout (four 16-lane groups with two packed pairs each) of 32-bit
// column words.
constexpr int kWaveBuf = 2 * 4 * 2 * RefStager<16>::kBuf;
constexpr int kNoRow = 0x7FFFFFFF;   // no cell found

// One sweep (forward, or reverse when REV) of the wave item
// order[first .. first+count), one pair per W-lane group, int32 arithmetic.
template <int W, int R, bool REV, int C = kChunk>
__device__ __forceinline__ void sweep_i32(const KParams& P, const SchemeLds& S, uint16_t* wbuf,
                                          int first, int count, int lane) {
    constexpr int G = 64 / W;
    using Stager = RefStager<W, C>;
    constexpr int reverse = REV ? 1 : 0;
    const int g = lane / W;
    const int l = lane % W;

    const int pair = g < count ? P.order[first + g] : -1;
    const PairJob J = load_job(P, pair, reverse);

    // wave-uniform step count: longest reference in the wavefront + ramp
    int mmax = J.m;
    for (int off = 32; off > 0; off >>= 1) mmax = imax(mmax, __shfl_xor(mmax, off));
    const int steps = __builtin_amdgcn_readfirstlane(mmax > 0 ? mmax + W - 1 : 0);

    uint16_t* buf = wbuf + g * Stager::kBuf;
    Stager stage;
    stage.load(P.refs, J, P.order, 0, l);

    // query rows of this lane (padding code below the query end)
    int a[R];
    {
        int raw[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            int i = l * R + r;
            i = i < J.n ? i : (J.n > 0 ? J.n - 1 : 0);
            const uint8_t* p = J.n > 0 ? P.queries + J.qbase + (int64_t)J.dir * i
                                       : reinterpret_cast<const uint8_t*>(P.order);
            raw[r] = *p;
        }
        const int A = S.alphabet[J.sid];
        int bad = -1;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            a[r] = checked(raw[r], l * R + r < J.n, A, kPad, bad);
        }
        stage.store(buf, J, A, 0, l, bad);
        set_flag(P.flags, kFlagBadResidue, (bad >= 0) & (P.validate != 0));
    }
    const int A = S.alphabet[J.sid];
    const int go = S.gap_open[J.sid];
    const int ge = S.gap_extend[J.sid];
    wave_lds_sync();

    // E[r] holds E of row r at the column the lane sweeps next: it is
    // advanced right after that row's H is computed, so H - o is never kept
    int H[R], E[R], best[R], bj[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { H[r] = 0; E[r] = 0; best[r] = 0; bj[r] = -1; }
    int Hlast = 0, Flast = 0, Hup_prev = 0;
    const uint16_t* rbl = buf + W - l;   // rbl[tt] = column t0 + tt - l

    // software pipeline: a row's score for the next step is read as soon as
    // its score for this step is used, and the matrix row offset of the
    // next step one step before that
    int sc[R];
    int bb_next = rbl[1];
    {
        const int bb0 = rbl[0];
#pragma unroll
        for (int r = 0; r < R; ++r) sc[r] = S.mat[bb0 + a[r]];
    }
    int bad = -1;
    int j = -l;
    for (int t0 = 0; t0 < steps; t0 += C) {
        const bool more = t0 + C < steps;
        if (more) stage.load(P.refs, J, P.order, t0 + C, l);
        const int tn = __builtin_amdgcn_readfirstlane(steps - t0 < C ? steps - t0 : C);
        for (int tt = 0; tt < tn; ++tt) {
            const int bb2 = rbl[tt + 2];
            const int Hup = shift_in_group<W>(Hlast);
            const int Fup = shift_in_group<W>(Flast);
            int diag = Hup_prev;
            Hup_prev = Hup;
            int Hmu = sat_sub(Hup, go);
            int F = Fup;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                F = imax(F - ge, Hmu);
                const int h = imax(imax(diag + sc[r], E[r]), F);
                sc[r] = S.mat[bb_next + a[r]];
                diag = H[r];
                H[r] = h;
                Hmu = sat_sub(h, go);
                E[r] = imax(E[r] - ge, Hmu);
                if (h > best[r]) { best[r] = h; bj[r] = j; }
            }
            Hlast = H[R - 1];
            Flast = F;
            bb_next = bb2;
            ++j;
        }
        if (more) {
            wave_lds_sync();
            stage.store(buf, J, A, t0 + C, l, bad);
            wave_lds_sync();
            // the two look-ahead reads of the next chunk's first steps were
            // taken from the old buffer; the new buffer holds the same
            // columns at entries W-l+0 and W-l+1, so re-read them
            bb_next = rbl[1];
            const int bb0 = rbl[0];
#pragma unroll
            for (int r = 0; r < R; ++r) sc[r] = S.mat[bb0 + a[r]];
        }
    }
    set_flag(P.flags, kFlagBadResidue, (bad >= 0) & (P.validate != 0));

    // best of this lane in row-major order, then of the group
    int lb = 0, li = -1, lj = -1;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (best[r] > lb) { lb = best[r]; li = l * R + r; lj = bj[r]; }
    for (int off = 1; off < W; off <<= 1) {
        const int ob = __shfl_xor(lb, off);
        const int oi = __shfl_xor(li, off);
        const int oj = __shfl_xor(lj, off);
        if (ob > lb || (ob == lb && oi < li)) { lb = ob; li = oi; lj = oj; }
    }
    if (l == 0 && pair >= 0) {
        if (!reverse) {
            sw_result res;
            if (lb > 0) { res.score = lb; res.q_start = -1; res.q_end = li; res.r_start = -1; res.r_end = lj; }
            else { res.score = 0; res.q_start = res.q_end = res.r_start = res.r_end = -1; }
            P.out[pair] = res;
        } else if (J.fwd_score > 0) {
            if (lb != J.fwd_score) {
                atomicOr(&P.flags[kFlagReverseMismatch], 1);
            } else {
                P.out[pair].q_start = J.fwd_qe - li;
                P.out[pair].r_start = J.fwd_re - lj;
            }
        }
    }
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// Columns are encoded as kColMax - j in the low 15 bits of a key; j ranges
// over -(W-1) .. kI16MaxRef + W - 2 for groups of up to 256 lanes, so
// kColMax - j stays within 0..32767.
constexpr int kColMax = 32767 - 255;
static_assert(kI16MaxRef + 256 - 2 <= kColMax, "column field of the keys overflows");

__device__ __forceinline__ uint32_t u32(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }
__device__ __forceinline__ u16x2 pk(uint32_t v) { return __builtin_bit_cast(u16x2, v); }

// max(x - y, 0) per 16-bit half
__device__ __forceinline__ u16x2 pk_sat_sub(u16x2 x, u16x2 y) { return __builtin_elementwise_sub_sat(x, y); }
// max of three per 16-bit half, for halves that are positive normal
// half-precision patterns (see above); one v_pk_maximum3_f16
__device__ __forceinline__ u16x2 pk_max3(u16x2 x, u16x2 y, u16x2 z) {
    const f16x2 a = __builtin_bit_cast(f16x2, x), b = __builtin_bit_cast(f16x2, y), c = __builtin_bit_cast(f16x2, z);
    return __builtin_bit_cast(u16x2, __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c));
}
__device__ __forceinline__ uint32_t umax3(uint32_t a, uint32_t b, uint32_t c) {
    const uint32_t m = a > b ? a : b;
    return m > c ? m : c;
}

// Scores of one step for both pairs: low half M[aA][bA], high half M[aB][bB],
// each sign-extended to 16 bits.
__device__ __forceinline__ u16x2 load_scores(const int8_t* mat, int addrA, int addrB) {
    s16x2 s;
    s.x = (short)mat[addrA];
    s.y = (short)mat[addrB];
    return __builtin_bit_cast(u16x2, s);
}

// One sweep of the wave item order[first .. first+count), two pairs per
// W-lane group packed into int16 halves.
template <int W, int R, bool REV, int C = kChunk>
__device__ __forceinline__ void sweep_i16(const KParams& P, const SchemeLds& S, uint16_t* wbuf,
                                          int first, int count, int lane) {
    using Stager = RefStager<W, C>;
    constexpr int reverse = REV ? 1 : 0;
    constexpr int RP = (R + 1) / 2;                 // row pairs per lane
    constexpr uint32_t K = kI16Bias;
    constexpr uint32_t K2 = K | (K << 16);
    const int g = lane / W;
    const int l = lane % W;

    const int slot = g * 2;
    const int pairA = slot < count ? P.order[first + slot] : -1;
    const int pairB = slot + 1 < count ? P.order[first + slot + 1] : -1;
    const PairJob JA = load_job(P, pairA, reverse);
    const PairJob JB = load_job(P, pairB, reverse);

    int mmax = imax(JA.m, JB.m);
    for (int off = 32; off > 0; off >>= 1) mmax = imax(mmax, __shfl_xor(mmax, off));
    const int steps = __builtin_amdgcn_readfirstlane(mmax > 0 ? mmax + W - 1 : 0);

    uint16_t* bufA = wbuf + (g * 2) * Stager::kBuf;
    uint16_t* bufB = bufA + Stager::kBuf;
    Stager stA, stB;
    stA.load(P.refs, JA, P.order, 0, l);
    stB.load(P.refs, JB, P.order, 0, l);

    // query rows: residue codes of A (low half) and B (high half)
    uint32_t apk[R];
    {
        int rawA[R], rawB[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = l * R + r;
            const int iA = i < JA.n ? i : (JA.n > 0 ? JA.n - 1 : 0);
            const int iB = i < JB.n ? i : (JB.n > 0 ? JB.n - 1 : 0);
            const uint8_t* pA = JA.n > 0 ? P.queries + JA.qbase + (int64_t)JA.dir * iA
                                         : reinterpret_cast<const uint8_t*>(P.order);
            const uint8_t* pB = JB.n > 0 ? P.queries + JB.qbase + (int64_t)JB.dir * iB
                                         : reinterpret_cast<const uint8_t*>(P.order);
            rawA[r] = *pA;
            rawB[r] = *pB;
        }
        const int AA = S.alphabet[JA.sid], AB = S.alphabet[JB.sid];
        int bad = -1;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t a = checked(rawA[r], l * R + r < JA.n, AA, kPad, bad);
            const uint32_t b = checked(rawB[r], l * R + r < JB.n, AB, kPad, bad);
            apk[r] = a | (b << 16);
        }
        stA.store(bufA, JA, AA, 0, l, bad);
        stB.store(bufB, JB, AB, 0, l, bad);
        set_flag(P.flags, kFlagBadResidue, (bad >= 0) & (P.validate != 0));
    }
    const int AA = S.alphabet[JA.sid], AB = S.alphabet[JB.sid];
    const u16x2 go2 = pk(cost16(S.gap_open[JA.sid]) | (cost16(S.gap_open[JB.sid]) << 16));
    const u16x2 ge2 = pk(cost16(S.gap_extend[JA.sid]) | (cost16(S.gap_extend[JB.sid]) << 16));
    const u16x2 zero = pk(K2);
    wave_lds_sync();

    // H[r], E[r] (biased): H of row r at the last column swept, E of row r
    // at the next column (advanced right after the row's H, so H - o is
    // never kept).  kA/kB: keys of row pairs.
    u16x2 H[R], E[R];
    uint32_t kA[RP], kB[RP];
#pragma unroll
    for (int r = 0; r < R; ++r) { H[r] = zero; E[r] = zero; }
#pragma unroll
    for (int p = 0; p < RP; ++p) { kA[p] = 0u; kB[p] = 0u; }
    uint32_t Hlast = K2, Flast = K2, Hup_prev = K2;
    const uint16_t* rblA = bufA + W - l;
    const uint16_t* rblB = bufB + W - l;

    // software pipeline: a row's score for the next step is read as soon as
    // its score for this step is used, and the matrix row offset of the
    // next step one step before that
    u16x2 sc[R];
    int bbA_next = rblA[1], bbB_next = rblB[1];
    {
        const int a0 = rblA[0], b0 = rblB[0];
#pragma unroll
        for (int r = 0; r < R; ++r) sc[r] = load_scores(S.mat, a0 + (int)(apk[r] & 0xFFFF), b0 + (int)(apk[r] >> 16));
    }
    int bad = -1;
    uint32_t jc = (uint32_t)(kColMax + l);   // kColMax - j with j = t - l
    for (int t0 = 0; t0 < steps; t0 += C) {
        const bool more = t0 + C < steps;
        if (more) {
            stA.load(P.refs, JA, P.order, t0 + C, l);
            stB.load(P.refs, JB, P.order, t0 + C, l);
        }
        const int tn = __builtin_amdgcn_readfirstlane(steps - t0 < C ? steps - t0 : C);
        for (int tt = 0; tt < tn; ++tt) {
            const int bbA2 = rblA[tt + 2];
            const int bbB2 = rblB[tt + 2];
            const u16x2 Hup = pk((uint32_t)shift_in_group<W>((int)Hlast, (int)K2));
            // F above the group is 0 (K); a zero fill gives the same F below
            // because of the max with K
            const u16x2 Fup = pk((uint32_t)shift_in_group_zero<W>((int)Flast));
            u16x2 diag = pk(Hup_prev);
            Hup_prev = u32(Hup);
            u16x2 Hmu = pk_sat_sub(Hup, go2);
            u16x2 F = Fup;
            const uint32_t jc1 = jc | 0x8000u;   // upper row of a pair wins ties
            uint32_t keyA0 = 0, keyB0 = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                F = pk_max3(pk_sat_sub(F, ge2), Hmu, zero);
                const u16x2 h = pk_max3(diag + sc[r], E[r], F);
                sc[r] = load_scores(S.mat, bbA_next + (int)(apk[r] & 0xFFFF), bbB_next + (int)(apk[r] >> 16));
                diag = H[r];
                H[r] = h;
                Hmu = pk_sat_sub(h, go2);
                E[r] = pk_max3(pk_sat_sub(E[r], ge2), Hmu, zero);
                const uint32_t hv = u32(h);
                if ((r & 1) == 0) {
                    keyA0 = (hv << 16) | jc1;
                    keyB0 = (hv & 0xFFFF0000u) | jc1;
                    if (r == R - 1) {
                        kA[r / 2] = kA[r / 2] > keyA0 ? kA[r / 2] : keyA0;
                        kB[r / 2] = kB[r / 2] > keyB0 ? kB[r / 2] : keyB0;
                    }
                } else {
                    kA[r / 2] = umax3(kA[r / 2], keyA0, (hv << 16) | jc);
                    kB[r / 2] = umax3(kB[r / 2], keyB0, (hv & 0xFFFF0000u) | jc);
                }
            }
            Hlast = u32(H[R - 1]);
            Flast = u32(F);
            bbA_next = bbA2;
            bbB_next = bbB2;
            --jc;
        }
        if (more) {
            wave_lds_sync();
            stA.store(bufA, JA, AA, t0 + C, l, bad);
            stB.store(bufB, JB, AB, t0 + C, l, bad);
            wave_lds_sync();
            bbA_next = rblA[1];
            bbB_next = rblB[1];
            const int a0 = rblA[0], b0 = rblB[0];
#pragma unroll
            for (int r = 0; r < R; ++r)
                sc[r] = load_scores(S.mat, a0 + (int)(apk[r] & 0xFFFF), b0 + (int)(apk[r] >> 16));
        }
    }
    set_flag(P.flags, kFlagBadResidue, (bad >= 0) & (P.validate != 0));

    // per pair: best of this lane in row-major order, then of the group
    // (scores unbiased; a best of 0 leaves the coordinates at -1)
    int lb[2] = {0, 0}, li[2] = {-1, -1}, lj[2] = {-1, -1};
#pragma unroll
    for (int p = 0; p < RP; ++p) {
        const uint32_t ks[2] = {kA[p], kB[p]};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int h = (int)(ks[q] >> 16) - (int)K;
            const int row = l * R + 2 * p + ((ks[q] & 0x8000u) ? 0 : 1);
            if (h > lb[q]) { lb[q] = h; li[q] = row; lj[q] = kColMax - (int)(ks[q] & 0x7FFFu); }
        }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        for (int off = 1; off < W; off <<= 1) {
            const int ob = __shfl_xor(lb[p], off);
            const int oi = __shfl_xor(li[p], off);
            const int oj = __shfl_xor(lj[p], off);
            if (ob > lb[p] || (ob == lb[p] && oi < li[p])) { lb[p] = ob; li[p] = oi; lj[p] = oj; }
        }
    }
    if (l == 0) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int pair = p == 0 ? pairA : pairB;
            const PairJob& J = p == 0 ? JA : JB;
            if (pair < 0) continue;
            if (!reverse) {
                sw_result res;
                if (lb[p] > 0) { res.score = lb[p]; res.q_start = -1; res.q_end = li[p]; res.r_start = -1; res.r_end = lj[p]; }
                else { res.score = 0; res.q_start = res.q_end = res.r_start = res.r_end = -1; }
                P.out[pair] = res;
            } else if (J.fwd_score > 0) {
                if (lb[p] != J.fwd_score) {
                    atomicOr(&P.flags[kFlagReverseMismatch], 1);
                } else {
                    P.out[pair].q_start = J.fwd_qe - li[p];
                    P.out[pair].r_start = J.fwd_re - lj[p];
                }
            }
        }
    }
}

// ---- drifted sweeps ---------------------------------------------------------
//
// The packed sweeps of the score sources whose bytes carry a bias (column
// words, the pair table, the query profile).  They compute the same H as
// sweep_i16 with fewer instructions per cell, in two ways.
//
// 1. Drift.  The value kept for a cell in row r of its lane at sweep step t is
//    H + z(r, t) with z(r, t) = K0 + e (r + t), where e is the gap extension
//    cost (one for all pairs of the launch: column-word schemes of several costs
//    have a launch each, DriftGroup) and t counts from the last renormalisation.  A gap extension moves one row down or one column (one
//    step) on and costs e, so in these terms E and F carry over unchanged:
//        E(r, t+1) = max(E(r, t), Hm(r, t), z(r, t+1))    Hm = H - (o - e)
//        F(r+1, t) = max(F(r, t), Hm(r, t))
//        H(r, t)   = max(Hm(r-1, t-1) + (M + o + e), E, F)
//    which saves the two saturating subtractions of every cell (8 packed
//    instructions become 6).  The score sources hold bytes M + o + e.  The
//    clamp at zero is z in E's maximum, a scalar (z is the same in every
//    lane); F needs none.  Padding rows and columns read byte 0, a score of
//    -(o + e).  A lane's last row is handed to the next lane's first with
//    e (R - 1) subtracted.  Every `period` steps the drift is taken off all
//    kept values, so z stays within [K0, kI16Bias] and a stored value never
//    exceeds H + kI16Bias, the range of sweep_i16.  Small values are
//    denormal half-precision patterns here; v_pk_maximum3_f16 compares and
//    returns them as they are (checked over all operand classes).
//
// 2. Tracking.  sweep_i16 spends 3 instructions per row and step on the
//    row-pair keys.
//    Forward: the drift is taken off Hm once per cell, and two maxima are
//    kept: per row over all steps (which gives the score and the upper row
//    that holds it), and per step over the lane's rows (which gives the first
//    column in which the lane reaches its best).  Two steps are folded into
//    one maximum of three, so a cell costs 2 instructions in place of 3.  The
//    per-step maxima are over values that also carry the row: the undrifting
//    add is a v_pk_mad_u16 that shifts the score up by k bits and puts a row
//    code below it, larger for upper rows, so that the maximum prefers the
//    upper row and the column found is that row's first.  That takes a score
//    bound of at most 0x7BFF >> k for the item's pairs (k = 3 for up to 8
//    rows per lane, 4 for up to 16).  A pair-table lane of more than 8 rows
//    keeps the maxima of its even and of its odd rows apart (kSets = 2), as
//    its scores leave fewer bits, and so do the lanes of cooperative groups
//    (kCoopSets: their long queries leave 2 bits, or 1 for the pair table).
//    Where the bound does not hold (queries of more than about 660 DNA or 520
//    protein residues) the code is left out: then the column may be too
//    small, when another row of the lane lower down holds the best score in
//    an earlier column (about 0.05% of related pairs).  The reverse sweep decides: the prefix box of a column that is
//    too small holds no cell of the best score, so no start is found, the
//    pair goes to the redo list and sw_redo_kernel looks for its end again.
//    Reverse: the score S is known, so a cell is looked at only when it can
//    hold S.  Per step one maximum over the lane's rows (rows 8 apart are
//    brought to the same drift) is compared with S, and only when some lane
//    may have reached it are the rows compared one by one.  That is about
//    0.6 instructions per cell in place of 3.

// Residues of the lane's query rows (the last one repeated past the query
// end), and how many of the rows lie within the query (<= 0: none).
template <int R>
__device__ __forceinline__ int load_rows(const KParams& P, const PairJob& J, int l, int (&raw)[R]) {
    const int rem = J.n - l * R;
    const uint8_t* base = J.n > 0 ? P.queries + J.qbase + (int64_t)J.dir * (l * R)
                                  : reinterpret_cast<const uint8_t*>(P.order);
    const int last = J.n > 0 ? rem - 1 : 0;
#pragma unroll
    for (int r = 0; r < R; ++r) raw[r] = base[J.n > 0 ? J.dir * (r < last ? r : last) : 0];
    return rem;
}

// Sums of wave-uniform values, as scalar instructions the compiler leaves in
// place: it otherwise keeps every multiple of e of an unrolled step in its own
// register and spills them.
__device__ __forceinline__ uint32_t s_add(uint32_t x, uint32_t y) {
    uint32_t r;
    asm("s_add_u32 %0, %1, %2" : "=s"(r) : "s"(__builtin_amdgcn_readfirstlane(x)), "s"(y) : "scc");
    return r;
}
__device__ __forceinline__ uint32_t s_sub(uint32_t x, uint32_t y) {
    uint32_t r;
    asm("s_sub_u32 %0, %1, %2" : "=s"(r) : "s"(__builtin_amdgcn_readfirstlane(x)), "s"(__builtin_amdgcn_readfirstlane(y)) : "scc");
    return r;
}

// x * y + a per 16-bit half, the low half of the wave-uniform a in both
__device__ __forceinline__ u16x2 pk_mad(u16x2 x, u16x2 y, uint32_t a) {
    u16x2 r;
    asm("v_pk_mad_u16 %0, %1, %2, %3 op_sel_hi:[1,1,0]" : "=v"(r) : "v"(x), "v"(y), "s"(a));
    return r;
}

// max per 16-bit half (integers)
__device__ __forceinline__ u16x2 pk_max(u16x2 x, u16x2 y) { return __builtin_elementwise_max(x, y); }

// Score sources of the drifted sweeps.  `rows` sets up the lane's query rows,
// `stage` writes a prepared chunk of the reference to LDS, `begin` reads what
// the chunk's first step needs.  Even steps use one set of column registers,
// odd steps another (PH), so that no register rotates: `step_begin`,
// `score(r)`, `row_done(r)` and `step_end` are called in that order within a
// step tt of the chunk.

// Column words: per reference column one 32-bit word with the bytes
// M[a][b] + o + e, a = 0..3, so a row's scores of both pairs are one
// v_perm_b32 of the pairs' words with the row's selector.
template <int W, int R, int C>
struct ColScores {
    using Stager = RefStager<W, C>;
    using Lds = SchemeLds;
    using Entry = uint32_t;
    static constexpr int kSide = 0;   // KParams::drift entry
    static constexpr int kSets = 1, kCoopSets = R > 4 ? 2 : 1;
    uint32_t sel[R];
    uint32_t ca[2], cb[2];

    __device__ __forceinline__ void check(const KParams& P, PairJob& J, int pair) const {
        if (pair < 0) J.sid = P.drift[kSide].sid;
    }
    __device__ __forceinline__ void rows(const KParams& P, const Lds& S, const PairJob& JA, const PairJob& JB, int l,
                                         int& bad) {
        // byte 0 picks pair A's score from its word (bytes 0..3 of the perm
        // input), byte 2 pair B's (bytes 4..7); bytes 1 and 3 are zero
        // (selector 0x0C), as is a row past the query end
        int rawA[R], rawB[R];
        const int remA = load_rows<R>(P, JA, l, rawA), remB = load_rows<R>(P, JB, l, rawB);
        const int AA = S.alphabet[JA.sid], AB = S.alphabet[JB.sid];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t a = checked(rawA[r], r < remA, AA, 0x0C, bad);
            const uint32_t b = checked(rawB[r], r < remB, AB, 0x0C - 4, bad) + 4;
            sel[r] = a | 0x0C00u | (b << 16) | 0x0C000000u;
        }
    }
    // upper bounds of the two pairs' scores (kRowBounds: from the group's rows)
    static constexpr bool kRowBounds = false;
    __device__ __forceinline__ void bounds(const KParams& P, const PairJob& JA, const PairJob& JB, int& a, int& b) const {
        a = (JA.n < JA.m ? JA.n : JA.m) * P.max_score[JA.sid];
        b = (JB.n < JB.m ? JB.n : JB.m) * P.max_score[JB.sid];
    }
    __device__ __forceinline__ void stage(const Stager& st, Entry* buf, const KParams&, const Lds& S, const PairJob& J,
                                          int t0, int l, int& bad) const {
        st.store_col(buf, J, S.alphabet[J.sid], S.colw[J.sid], t0, l, bad);
    }
    __device__ __forceinline__ void begin(const Entry* rA, const Entry* rB) {
        ca[0] = rA[0]; cb[0] = rB[0];
        ca[1] = rA[1]; cb[1] = rB[1];
    }
    template <int PH> __device__ __forceinline__ void step_begin(const Entry*, const Entry*, int) {}
    template <int PH> __device__ __forceinline__ u16x2 score(int r) const {
        return pk(__builtin_amdgcn_perm(cb[PH], ca[PH], sel[r]));
    }
    template <int PH> __device__ __forceinline__ void row_done(int) {}
    template <int PH> __device__ __forceinline__ void step_end(const Entry* rA, const Entry* rB, int tt) {
        ca[PH] = rA[tt + 2];
        cb[PH] = rB[tt + 2];
    }
};

// Pair table of scheme P.ptab_sid (alphabets of up to 24 residues): entry
// [(x D + y) D + b] holds the bytes M[x][b] + o + e and M[y][b] + o + e for
// two consecutive query rows with residues x, y (D = alphabet + 1; code
// D - 1 pads rows past the query end and columns outside the reference with
// 0).  A lane's row pair p reads both of its scores for one column with a
// single 16-bit LDS load at rc[p] + 2 b, where rc[p] is a per-row-pair
// constant: one address add and one load per two rows and pair; one
// v_perm_b32 per row then places pair A's score in the low half and pair B's
// in the high half.  A row pair's scores of the next step are loaded as soon
// as the pair has used the current ones.
template <int W, int R, int C>
struct PtabScores {
    using Stager = RefStager<W, C>;
    using Lds = PtabLds;
    using Entry = uint16_t;
    static constexpr int kSide = 1;
    static constexpr int kSets = R > 8 ? 2 : 1, kCoopSets = R > 4 ? 4 : R > 2 ? 2 : 1;
    static constexpr int RP = (R + 1) / 2;
    // Up to 14 rows per lane pairs A and B keep their scores in separate
    // registers (one v_perm_b32 per row reads both); above that the two
    // loads fill the halves of one register, which costs one more v_perm_b32
    // per row pair but keeps the kernel within 256 registers, i.e. two
    // wavefronts per SIMD instead of one.
    static constexpr bool kSplit = R <= 14;
    // byte offsets of a row pair's table rows, ((x D + y) D) * 2, for pair A
    // (low half) and pair B (high half); both are below 2 D^3 <= 2^15
    uint32_t rc[RP];
    uint32_t uA[RP], uB[kSplit ? RP : 1];
    uint32_t xa[2], xb[2];
    const uint8_t* tab;
    int sumA, sumB;   // scores of this lane's rows at their best
    static constexpr bool kRowBounds = true;

    __device__ __forceinline__ void check(const KParams& P, PairJob& J, int pair) const {
        // every pair of a pair-table item uses the table's scheme; anything
        // else is an internal error, swept as an empty pair
        const bool other = pair >= 0 && J.sid != P.ptab_sid;
        set_flag(P.flags, kFlagInternal, other);
        J.n = other ? 0 : J.n;
        J.m = other ? 0 : J.m;
        J.fwd_score = other ? 0 : J.fwd_score;
        J.sid = P.ptab_sid;
    }
    __device__ __forceinline__ void rows(const KParams& P, const Lds& S, const PairJob& JA, const PairJob& JB, int l,
                                         int& bad) {
        tab = reinterpret_cast<const uint8_t*>(S.tab);
        const int D = P.ptab_dim, A = D - 1;
        int rawA[R], rawB[R];
        const int remA = load_rows<R>(P, JA, l, rawA), remB = load_rows<R>(P, JB, l, rawB);
        int xA[2 * RP], xB[2 * RP];
        sumA = sumB = 0;
#pragma unroll
        for (int r = 0; r < 2 * RP; ++r) {
            if (r >= R) {   // the row below an odd lane's last
                xA[r] = xB[r] = D - 1;
                continue;
            }
            const int ra = rawA[r < R ? r : 0], rb = rawB[r < R ? r : 0];
            xA[r] = checked(ra, r < remA, A, D - 1, bad);
            xB[r] = checked(rb, r < remB, A, D - 1, bad);
            sumA += S.row_max[xA[r]];
            sumB += S.row_max[xB[r]];
        }
#pragma unroll
        for (int p = 0; p < RP; ++p)
            rc[p] = (uint32_t)((xA[2 * p] * D + xA[2 * p + 1]) * D * 2) |
                    ((uint32_t)((xB[2 * p] * D + xB[2 * p + 1]) * D * 2) << 16);
    }
    __device__ __forceinline__ void stage(const Stager& st, Entry* buf, const KParams& P, const Lds&, const PairJob& J,
                                          int t0, int l, int& bad) const {
        st.store_ptab(buf, J, P.ptab_dim - 1, P.ptab_dim, t0, l, bad);
    }
    __device__ __forceinline__ void bounds(const KParams&, const PairJob&, const PairJob&, int& a, int& b) const {
        a = sumA;
        b = sumB;
        for (int off = 1; off < W; off <<= 1) {
            a += __shfl_xor(a, off);
            b += __shfl_xor(b, off);
        }
    }
    __device__ __forceinline__ void load_pair(int p, uint32_t ca, uint32_t cb) {
        const uint32_t a = *reinterpret_cast<const uint16_t*>(tab + (rc[p] & 0xFFFFu) + ca);
        const uint32_t b = *reinterpret_cast<const uint16_t*>(tab + (rc[p] >> 16) + cb);
        if constexpr (kSplit) {
            uA[p] = a;
            uB[p] = b;
        } else {
            uA[p] = __builtin_amdgcn_perm(b, a, 0x05040100u);
        }
    }
    __device__ __forceinline__ void begin(const Entry* rA, const Entry* rB) {
        xa[0] = rA[0]; xb[0] = rB[0];
        xa[1] = rA[1]; xb[1] = rB[1];
#pragma unroll
        for (int p = 0; p < RP; ++p) load_pair(p, xa[0], xb[0]);
    }
    template <int PH> __device__ __forceinline__ void step_begin(const Entry* rA, const Entry* rB, int tt) {
        // this step's scores are loaded already: its offsets make way for
        // those two steps ahead
        xa[PH] = rA[tt + 2];
        xb[PH] = rB[tt + 2];
    }
    template <int PH> __device__ __forceinline__ u16x2 score(int r) const {
        const int p = r / 2;
        if constexpr (kSplit)
            return pk(__builtin_amdgcn_perm(uB[p], uA[p], (r & 1) ? 0x0C050C01u : 0x0C040C00u));
        else
            return pk(__builtin_amdgcn_perm(uA[p], uA[p], (r & 1) ? 0x0C030C01u : 0x0C020C00u));
    }
    template <int PH> __device__ __forceinline__ void row_done(int r) {
        if ((r & 1) == 1 || r == R - 1) load_pair(r / 2, xa[PH ^ 1], xb[PH ^ 1]);
    }
    template <int PH> __device__ __forceinline__ void step_end(const Entry*, const Entry*, int) {}
};

// Query profile (the forward pass of a database search, where every pair
// aligns the same query): byte ((b W + l) Rp + r) is M[a_i][b] + o + e for
// row i = l R + r of lane l (0 past the query end, and for the padding code
// b = D - 1), with Rp = R rounded up to whole dwords.  A lane reads its R
// rows' scores for one reference residue as Rp/4 consecutive dwords at one
// address (one add per pair and step), and one v_perm_b32 per row places
// pair A's score in the low half and pair B's in the high half.
template <int W, int R>
struct QprofLds {
    static constexpr int RD = (R + 3) / 4;          // profile dwords per lane and residue
    static constexpr int kRowBytes = W * RD * 4;    // profile bytes per residue
    uint8_t prof[kPtabMaxDim * kRowBytes];
    int32_t gap_open[SW_MAX_SCHEMES];
    int32_t bound;   // the query's score against itself at best
};

template <int W, int R, int C>
struct QprofScores {
    using Stager = RefStager<W, C>;
    using Lds = QprofLds<W, R>;
    using Entry = uint16_t;
    static constexpr int kSide = 1;
    static constexpr int kSets = R > 8 ? 2 : 1, kCoopSets = 1;   // (never cooperative)
    static constexpr int RD = Lds::RD;
    uint32_t dA[RD], dB[RD];
    uint32_t xa[2], xb[2];
    const uint8_t* lprof;   // this lane's rows of residue 0
    int bound;
    static constexpr bool kRowBounds = false;

    __device__ __forceinline__ void check(const KParams& P, PairJob& J, int pair) const {
        // every pair aligns the profiled query with the profile's scheme
        const bool other = pair >= 0 && (J.sid != P.ptab_sid || J.n != P.qprof_n);
        set_flag(P.flags, kFlagInternal, other);
        J.n = other ? 0 : J.n;
        J.m = other ? 0 : J.m;
        J.sid = P.ptab_sid;
    }
    __device__ __forceinline__ void rows(const KParams&, const Lds& S, const PairJob&, const PairJob&, int l, int&) {
        lprof = S.prof + l * RD * 4;
        bound = S.bound;
    }
    __device__ __forceinline__ void bounds(const KParams&, const PairJob&, const PairJob&, int& a, int& b) const {
        a = b = bound;
    }
    __device__ __forceinline__ void stage(const Stager& st, Entry* buf, const KParams& P, const Lds&, const PairJob& J,
                                          int t0, int l, int& bad) const {
        st.store_qprof(buf, J, P.ptab_dim - 1, P.ptab_dim, Lds::kRowBytes, t0, l, bad);
    }
    __device__ __forceinline__ void begin(const Entry* rA, const Entry* rB) {
        xa[0] = rA[0]; xb[0] = rB[0];
        xa[1] = rA[1]; xb[1] = rB[1];
#pragma unroll
        for (int k = 0; k < RD; ++k) {
            dA[k] = *reinterpret_cast<const uint32_t*>(lprof + xa[0] + 4 * k);
            dB[k] = *reinterpret_cast<const uint32_t*>(lprof + xb[0] + 4 * k);
        }
    }
    template <int PH> __device__ __forceinline__ void step_begin(const Entry* rA, const Entry* rB, int tt) {
        xa[PH] = rA[tt + 2];
        xb[PH] = rB[tt + 2];
    }
    template <int PH> __device__ __forceinline__ u16x2 score(int r) const {
        const uint32_t sel = (uint32_t)(r % 4) | 0x0C00u | ((uint32_t)(4 + r % 4) << 16) | 0x0C000000u;
        return pk(__builtin_amdgcn_perm(dB[r / 4], dA[r / 4], sel));
    }
    template <int PH> __device__ __forceinline__ void row_done(int r) {
        if (r % 4 == 3 || r == R - 1) {
            dA[r / 4] = *reinterpret_cast<const uint32_t*>(lprof + xa[PH ^ 1] + 4 * (r / 4));
            dB[r / 4] = *reinterpret_cast<const uint32_t*>(lprof + xb[PH ^ 1] + 4 * (r / 4));
        }
    }
    template <int PH> __device__ __forceinline__ void step_end(const Entry*, const Entry*, int) {}
};

// Pairs whose reverse sweep found no start go to the redo list (see above).
__device__ __forceinline__ void push_redo(const KParams& P, int pair) {
    const int k = atomicAdd(&P.meta[kMetaRedo], 1);
    if (k >= 0 && k < P.n_pairs) P.redo[k] = pair;
    else atomicOr(&P.flags[kFlagInternal], 1);
}

// Exchange between the four wavefronts of a cooperative group (sw_coop.h).
// ring[w][j % 128]: H - (o - e) and F of the row above wavefront w's first
// row at column j, without drift; ring[0][0] is the matrix's top boundary.
struct CoopX {
    uint2 ring[kWavesPerBlock][128];
    uint2 dump[128 + 64];                 // where the lanes that hand nothing on write
    int32_t res[kWavesPerBlock][2][3];    // per wavefront and pair: best, row, column
    int32_t item;
};

// One sweep of two jobs per W-lane group packed into int16 halves, scores from
// Src.  Forward, the results of pairs A and B (-1: none) are written; REV looks
// for the row-major-first cell that holds a job's score (J.fwd_score, 0: none)
// and calls found(row, col) in every lane, row kNoRow without one.  With COOP
// the four wavefronts of the workgroup sweep one item as a group of 256 lanes:
// this wavefront is number `wave` of it (see sw_coop.h), W is 64.
template <class Src, int W, int R, bool REV, int C, bool COOP, class Found>
__device__ __forceinline__ void sweep_jobs(const KParams& P, const typename Src::Lds& S, uint16_t* wbuf,
                                           PairJob JA, PairJob JB, int pairA, int pairB, int lane, CoopX* X, int wave,
                                           Found&& found) {
    static_assert(!COOP || (W == 64 && C == 128), "a cooperative group is four 64-lane wavefronts");
    using Stager = RefStager<W, C>;
    using Entry = typename Src::Entry;
    constexpr uint32_t K2 = (uint32_t)kI16Bias * 0x10001u;
    const int g = lane / W;
    const int l = lane % W;
    const int lr = COOP ? 64 * wave + l : l;   // lane within the pair's group: rows lr * R ..
    Src src;
    src.check(P, JA, pairA);
    src.check(P, JB, pairB);

    // wave-uniform step count, even (steps run in twos; a step past the last
    // reads padding columns)
    int mmax = imax(JA.m, JB.m);
    for (int off = 32; off > 0; off >>= 1) mmax = imax(mmax, __shfl_xor(mmax, off));
    const int steps = __builtin_amdgcn_readfirstlane(mmax > 0 ? (mmax + W) & ~1 : 0);

    Entry* bufA = reinterpret_cast<Entry*>(wbuf) + (g * 2) * Stager::kBuf;
    Entry* bufB = bufA + Stager::kBuf;
    Stager stA, stB;
    stA.load(P.refs, JA, P.order, 0, l);
    stB.load(P.refs, JB, P.order, 0, l);
    int bad = -1;
    src.rows(P, S, JA, JB, lr, bad);
    src.stage(stA, bufA, P, S, JA, 0, l, bad);
    src.stage(stB, bufB, P, S, JB, 0, l, bad);

    const uint32_t e = (uint32_t)P.drift[Src::kSide].e;
    const int period = P.drift[Src::kSide].period;       // even, at least 2
    const uint32_t e2 = __builtin_amdgcn_readfirstlane(e * 0x10001u), e8 = 8u * e2;
    const uint32_t goA = (uint32_t)S.gap_open[JA.sid], goB = (uint32_t)S.gap_open[JB.sid];
    const uint32_t cAB = (goA - e) | ((goB - e) << 16);   // o - e of both pairs
    const u16x2 c2 = pk(cAB);
    // z(r, t) = z0 + e2 (r + t); the largest one used is z(R, period)
    const uint32_t z0 = K2 - e2 * (uint32_t)(R + period + 1);
    const u16x2 lift = pk(e2 * (uint32_t)(R - 1));        // a lane's last row, as seen from the next lane
    wave_lds_sync();

    // Hm[r]: H - (o - e) of row r at the last step; E[r]: E of row r at the
    // next step (both drifted); the state before step 0 is H = 0 everywhere
    u16x2 Hm[R], E[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        Hm[r] = pk(z0 + e2 * (uint32_t)r - e2) - c2;
        E[r] = pk(z0 + e2 * (uint32_t)r);
    }
    u16x2 Hlast = Hm[R - 1], Flast = Hlast;
    u16x2 Hup_prev = pk(z0 - 2u * e2) - c2;
    // forward: v = ((H - (o - e) + x) << k) + row code, its largest per row,
    // and per pair and set of rows the key (largest v of a step << 16) |
    // (kColMax - column), largest first
    constexpr int kSets = REV ? 1 : COOP ? Src::kCoopSets : Src::kSets;
    constexpr int kQ = (R + kSets - 1) / kSets;      // rows of a set
    constexpr int kCode = kQ <= 1 ? 0 : kQ <= 2 ? 1 : kQ <= 4 ? 2 : kQ <= 8 ? 3 : kQ <= 16 ? 4 : 5;
    u16x2 best[REV ? 1 : R];
    uint32_t kA[kSets], kB[kSets];
    const int x = P.drift[Src::kSide].x;
    int k = 0;
    if constexpr (!REV) {
        int a, b;
        src.bounds(P, JA, JB, a, b);
        if constexpr (COOP && Src::kRowBounds) {
            // the bounds of the wavefronts' rows add up
            X->res[wave][0][0] = a;
            X->res[wave][1][0] = b;
            __syncthreads();
            a = b = 0;
            for (int w = 0; w < kWavesPerBlock; ++w) {
                a += X->res[w][0][0];
                b += X->res[w][1][0];
            }
        }
        a = imax(a + x - (int)(goA - e), b + x - (int)(goB - e));
        k = __builtin_amdgcn_ballot_w64(((a + 1) << kCode) > 0x7C00) == 0 ? kCode : 0;
    }
    const u16x2 scale = pk(0x10001u << k);
    const uint32_t ek = __builtin_amdgcn_readfirstlane(e << k);
    const uint32_t dcode = __builtin_amdgcn_readfirstlane(k > 0 ? 1 : 0);   // code step from one row of a set to the next
    // undrifting term of row 0 at step 0
    const uint32_t a0 = __builtin_amdgcn_readfirstlane((((uint32_t)x - (z0 & 0xFFFFu)) << k) + (k > 0 ? kQ - 1 : 0));
    // reverse: a cell holds S when Hm >= z + thr + 1; row and column found
    u16x2 thr = pk(0);
    int rowA = R, rowB = R, colA = 0, colB = 0;   // row within the lane
    if constexpr (REV) {
        const uint32_t tA = JA.fwd_score > 0 ? (uint32_t)(JA.fwd_score - (int)(goA - e) - 1) & 0xFFFFu : 0x7C00u;
        const uint32_t tB = JB.fwd_score > 0 ? (uint32_t)(JB.fwd_score - (int)(goB - e) - 1) & 0xFFFFu : 0x7C00u;
        thr = pk(tA | (tB << 16));
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) best[r] = pk(0);
#pragma unroll
        for (int q = 0; q < kSets; ++q) kA[q] = kB[q] = 0;
    }
    const Entry* rA = bufA + W - l;   // rA[tt]: entry of column t0 + tt - l
    const Entry* rB = bufB + W - l;
    uint32_t jc = (uint32_t)(kColMax + l);   // kColMax - j with j = t - l

    // cooperative groups: blocks of `block` steps between workgroup barriers.
    // Wavefront w starts `lag` blocks after the one above it, whose last lane
    // is 63 columns behind its first: what a block reads was written in
    // earlier ones.
    const int block = COOP && period > 32 ? 32 : period;
    const int lag = 63 / block + 2;
    const int ring_mask = wave > 0 ? 127 : 0;
    const int cols = __builtin_amdgcn_readfirstlane(mmax);
    uint2 above = make_uint2(0, 0);
    uint2* below = nullptr;
    if constexpr (COOP) {
        below = l == 63 && wave + 1 < kWavesPerBlock ? X->ring[wave + 1] : X->dump + l;
        if (wave == 0) {
            const uint32_t none = u32(pk(0) - c2);
            X->ring[0][0] = make_uint2(none, none);
            wave_lds_sync();
        }
        // (the barriers also show the top boundary to the wavefronts below)
        for (int q = 0; q < lag * wave; ++q) __syncthreads();
        above = X->ring[wave][0];
    }

    uint32_t zs[R + 2];   // z(r, t) of the even step t, for it and the odd step after it
    // Step tt of the chunk; zt = z(0, t).  Odd steps (PH = 1) also track the
    // even step before them (forward); at is that step's undrifting term.
    auto step = [&](auto phase, int t0, int tt, uint32_t zt, uint32_t at) {
        constexpr int PH = decltype(phase)::value;
        src.template step_begin<PH>(rA, rB, tt);
        // the row above the lane's block; above the group it is the matrix's
        // top boundary, H = 0 (z of row -1) and no F
        const uint32_t zup = s_sub(zt, e2);
        u16x2 Hup, F;
        if constexpr (COOP) {
            // from the wavefront above, or the top boundary
            Hup = pk((uint32_t)shift_in_group<W>((int)u32(Hlast - lift), (int)u32(pk(above.x) + pk(zup))));
            F = pk((uint32_t)shift_in_group<W>((int)u32(Flast - lift), (int)u32(pk(above.y) + pk(zup))));
            // (columns past the reference are not handed on)
            above = t0 + tt + 1 < cols ? X->ring[wave][(tt + 1) & ring_mask] : X->ring[0][0];
        } else {
            const u16x2 top = pk(zup) - c2;
            Hup = pk((uint32_t)shift_in_group<W>((int)u32(Hlast - lift), (int)u32(top)));
            F = pk((uint32_t)shift_in_group_zero<W>((int)u32(Flast - lift)));
        }
        u16x2 diag = Hup_prev;
        Hup_prev = Hup;
        u16x2 Hmu = Hup;
        if constexpr (PH == 0 || R > 16) {   // (more rows would not leave enough scalar registers)
            zs[0] = PH == 0 ? zt : zup;
#pragma unroll
            for (int r = 1; r < R + 2; ++r) zs[r] = s_add(zs[r - 1], e2);
        }
        uint32_t a = at;
        u16x2 me[kSets], mo[kSets], pe[kSets], po[kSets], f = pk(0), pn = pk(0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            F = pk_max(F, Hmu);
            const u16x2 h = pk_max3(diag + src.template score<PH>(r), E[r], F);
            const u16x2 old = Hm[r];
            const u16x2 hm = h - c2;
            diag = old;
            Hm[r] = hm;
            Hmu = hm;
            E[r] = pk_max3(E[r], hm, pk(zs[r + 1 + PH]));
            if constexpr (REV) {
                if (r % 8 == 0 && r > 0) f = f + pk(e8);
                if (r == 0) f = hm;
                else if ((r & 1) == 0) pn = hm;
                else f = r == 1 ? pk_max(f, hm) : pk_max3(f, pn, hm);
                if ((r & 1) == 0 && r == R - 1 && r > 0) f = pk_max(f, hm);
            } else if constexpr (PH == 1) {
                const u16x2 ue = pk_mad(old, scale, a);
                a = s_sub(a, ek);
                const u16x2 uo = pk_mad(hm, scale, a);
                if (r % kSets == kSets - 1) a = s_sub(a, dcode);
                best[r] = pk_max3(best[r], ue, uo);
                const int q = r / kSets, g2 = r % kSets;
                const bool last = r + kSets >= R;   // of its set
                if ((q & 1) == 0) {
                    pe[g2] = ue;
                    po[g2] = uo;
                    if (last) {
                        me[g2] = q == 0 ? ue : pk_max(me[g2], ue);
                        mo[g2] = q == 0 ? uo : pk_max(mo[g2], uo);
                    }
                } else {
                    me[g2] = q == 1 ? pk_max(pe[g2], ue) : pk_max3(me[g2], pe[g2], ue);
                    mo[g2] = q == 1 ? pk_max(po[g2], uo) : pk_max3(mo[g2], po[g2], uo);
                }
            }
            src.template row_done<PH>(r);
        }
        Hlast = Hm[R - 1];
        Flast = F;
        src.template step_end<PH>(rA, rB, tt);
        if constexpr (COOP) {
            // the last lane hands its last row on: column t - 63, drift off
            const u16x2 zl = pk(zs[R - 1 + PH]);
            below[(tt + 65) & 127] = make_uint2(u32(Hlast - zl), u32(Flast - zl));
        }
        if constexpr (REV) {
            // the last group of 8 rows starts at row 8 * ((R - 1) / 8)
            uint32_t zg = zt;
#pragma unroll
            for (int q = 0; q < (R - 1) / 8; ++q) zg = s_add(zg, e8);
            const u16x2 over = pk_sat_sub(f, thr + pk(zg));
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(u32(over) != 0) != 0, 0)) {
                uint32_t any = 0, zr = zt;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    any |= u32(pk_sat_sub(Hm[r], thr + pk(zr)));
                    zr = s_add(zr, e2);
                }
                if (__builtin_amdgcn_ballot_w64(any != 0) != 0) {
                    int hitA = R, hitB = R;
#pragma unroll
                    for (int r = R - 1; r >= 0; --r) {
                        zr = s_sub(zr, e2);
                        const uint32_t w = u32(pk_sat_sub(Hm[r], thr + pk(zr)));
                        hitA = (w & 0xFFFFu) ? r : hitA;
                        hitB = (w >> 16) ? r : hitB;
                    }
                    const int j = kColMax - (int)jc;
                    colA = hitA < rowA ? j : colA;
                    colB = hitB < rowB ? j : colB;
                    rowA = hitA < rowA ? hitA : rowA;
                    rowB = hitB < rowB ? hitB : rowB;
                }
            }
            --jc;
        } else if constexpr (PH == 1) {
#pragma unroll
            for (int q = 0; q < kSets; ++q) {
                if (q >= R) continue;   // (a set has at least one row)
                const uint32_t ve = u32(me[q]), vo = u32(mo[q]);
                kA[q] = umax3(kA[q], (ve << 16) | jc, (vo << 16) | (jc - 1));
                kB[q] = umax3(kB[q], (ve & 0xFFFF0000u) | jc, (vo & 0xFFFF0000u) | (jc - 1));
            }
            jc -= 2;
        }
    };
    for (int t0 = 0; t0 < steps; t0 += C) {
        const bool more = t0 + C < steps;
        if (more) {
            stA.load(P.refs, JA, P.order, t0 + C, l);
            stB.load(P.refs, JB, P.order, t0 + C, l);
        }
        const int tn = __builtin_amdgcn_readfirstlane(steps - t0 < C ? steps - t0 : C);
        src.begin(rA, rB);
        for (int s0 = 0; s0 < tn; s0 += block) {
            const int s1 = tn - s0 < block ? tn : s0 + block;
            uint32_t zt = z0, at = a0;
            for (int tt = s0; tt < s1; tt += 2) {
                step(std::integral_constant<int, 0>{}, t0, tt, zt, at);
                step(std::integral_constant<int, 1>{}, t0, tt + 1, zt + e2, at);
                zt += 2u * e2;
                at -= 2u * ek;
            }
            // renormalise: the next step counts as step 0 again
            const u16x2 back = pk(e2 * (uint32_t)(s1 - s0));
#pragma unroll
            for (int r = 0; r < R; ++r) {
                Hm[r] = Hm[r] - back;
                E[r] = E[r] - back;
            }
            Hlast = Hm[R - 1];
            Flast = Flast - back;
            Hup_prev = Hup_prev - back;
            if constexpr (COOP) __syncthreads();
        }
        if (more) {
            wave_lds_sync();
            src.stage(stA, bufA, P, S, JA, t0 + C, l, bad);
            src.stage(stB, bufB, P, S, JB, t0 + C, l, bad);
            wave_lds_sync();
        }
    }
    set_flag(P.flags, kFlagBadResidue, (bad >= 0) & (P.validate != 0));
    if constexpr (COOP)
        for (int q = 0; q < lag * (kWavesPerBlock - 1 - wave); ++q) __syncthreads();

    if constexpr (REV) {
        int row[2] = {rowA < R ? lr * R + rowA : kNoRow, rowB < R ? lr * R + rowB : kNoRow}, col[2] = {colA, colB};
#pragma unroll
        for (int p = 0; p < 2; ++p)
            for (int off = 1; off < W; off <<= 1) {
                const int oi = __shfl_xor(row[p], off);
                const int oj = __shfl_xor(col[p], off);
                col[p] = oi < row[p] ? oj : col[p];
                row[p] = oi < row[p] ? oi : row[p];
            }
        if constexpr (COOP) {
            // upper wavefronts hold upper rows
#pragma unroll
            for (int p = 0; p < 2; ++p) { X->res[wave][p][1] = row[p]; X->res[wave][p][2] = col[p]; }
            __syncthreads();
#pragma unroll
            for (int p = 0; p < 2; ++p)
                for (int w = kWavesPerBlock - 1; w >= 0; --w)
                    if (X->res[w][p][1] != kNoRow) { row[p] = X->res[w][p][1]; col[p] = X->res[w][p][2]; }
        }
        found(row, col);
    } else {
        // per pair: best of this lane, its upper row, and the lane's first
        // column that reaches it; then the group's, upper rows first
        const int zero[2] = {x - (int)(goA - e), x - (int)(goB - e)};
        int lb[2] = {0, 0}, li[2] = {-1, -1}, lj[2] = {-1, -1};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t b = u32(best[r]);
            const int h[2] = {(int)((b & 0xFFFFu) >> k) - zero[0], (int)(b >> 16 >> k) - zero[1]};
            const uint32_t key[2] = {kA[r % kSets], kB[r % kSets]};
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                li[p] = h[p] > lb[p] ? r : li[p];
                lj[p] = h[p] > lb[p] ? (int)key[p] : lj[p];
                lb[p] = h[p] > lb[p] ? h[p] : lb[p];
            }
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            lj[p] = lb[p] > 0 ? kColMax - (lj[p] & 0x7FFF) : -1;
            li[p] = lb[p] > 0 ? lr * R + li[p] : -1;
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            for (int off = 1; off < W; off <<= 1) {
                const int ob = __shfl_xor(lb[p], off);
                const int oi = __shfl_xor(li[p], off);
                const int oj = __shfl_xor(lj[p], off);
                const bool take = (ob > lb[p]) | ((ob == lb[p]) & (oi < li[p]));
                lb[p] = take ? ob : lb[p];
                li[p] = take ? oi : li[p];
                lj[p] = take ? oj : lj[p];
            }
        }
        if constexpr (COOP) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                X->res[wave][p][0] = lb[p];
                X->res[wave][p][1] = li[p];
                X->res[wave][p][2] = lj[p];
            }
            __syncthreads();
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                lb[p] = 0;
                for (int w = 0; w < kWavesPerBlock; ++w)
                    if (X->res[w][p][0] > lb[p]) {
                        lb[p] = X->res[w][p][0];
                        li[p] = X->res[w][p][1];
                        lj[p] = X->res[w][p][2];
                    }
            }
        }
        if (lr == 0) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int pair = p == 0 ? pairA : pairB;
                if (pair < 0) continue;
                sw_result res;
                if (lb[p] > 0) { res.score = lb[p]; res.q_start = -1; res.q_end = li[p]; res.r_start = -1; res.r_end = lj[p]; }
                else { res.score = 0; res.q_start = res.q_end = res.r_start = res.r_end = -1; }
                P.out[pair] = res;
            }
        }
    }
}

// The sweep of the wave item order[first .. first+count): its pairs, forward or,
// REV, back from their ends.
template <class Src, int W, int R, bool REV, int C, bool COOP = false>
__device__ __forceinline__ void sweep_drift(const KParams& P, const typename Src::Lds& S, uint16_t* wbuf, int first,
                                            int count, int lane, CoopX* X = nullptr, int wave = 0) {
    const int slot = lane / W * 2;
    int pairA = slot < count ? P.order[first + slot] : -1;
    int pairB = slot + 1 < count ? P.order[first + slot + 1] : -1;
    PairJob JA = load_job(P, pairA, REV ? 1 : 0);
    PairJob JB = load_job(P, pairB, REV ? 1 : 0);
    if constexpr (Src::kSide == 0) {
        keep_group(P, JA, pairA);
        keep_group(P, JB, pairB);
    }
    sweep_jobs<Src, W, R, REV, C, COOP>(P, S, wbuf, JA, JB, pairA, pairB, lane, X, wave,
                                        [&](const int (&row)[2], const int (&col)[2]) {
        if ((COOP && wave > 0) || lane % W != 0) return;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int pair = p == 0 ? pairA : pairB;
            const PairJob& J = p == 0 ? JA : JB;
            if (pair < 0 || J.fwd_score <= 0) continue;
            if (row[p] == kNoRow) {
                push_redo(P, pair);
            } else {
                P.out[pair].q_start = J.fwd_qe - row[p];
                P.out[pair].r_start = J.fwd_re - col[p];
            }
        }
    });
}

}  // namespace sw
