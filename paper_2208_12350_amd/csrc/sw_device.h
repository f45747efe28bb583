// sw_device.h -- device-side helpers shared by the gfx950 sweep kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sw_internal.h"

namespace sw {

template <int W>
__device__ __forceinline__ int shift_in_group(int x, int fill = 0) {
    // Lane l receives lane l-1's value; the first lane of each W-lane group
    // receives `fill`.  row_shr:1 shifts within 16-lane rows, wave_shr:1
    // across the whole wavefront; with bound_ctrl off, a lane with no source
    // keeps the `old` operand.  32-lane groups take the wave shift and
    // select `fill` for lane 32 (its source, lane 31, belongs to the other
    // group).
    if constexpr (W == 16) {
        return __builtin_amdgcn_update_dpp(fill, x, 0x111, 0xF, 0xF, false);
    } else if constexpr (W == 32) {
        const int y = __builtin_amdgcn_update_dpp(fill, x, 0x138, 0xF, 0xF, false);
        return (__lane_id() & 31) ? y : fill;
    } else {
        static_assert(W == 64, "W must be 16, 32 or 64");
        return __builtin_amdgcn_update_dpp(fill, x, 0x138, 0xF, 0xF, false);
    }
}

// shift_in_group with a zero fill: bound_ctrl writes the zero, so no fill
// register has to be set up.
template <int W>
__device__ __forceinline__ int shift_in_group_zero(int x) {
    if constexpr (W == 16) {
        return __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);
    } else if constexpr (W == 32) {
        const int y = __builtin_amdgcn_update_dpp(0, x, 0x138, 0xF, 0xF, true);
        return (__lane_id() & 31) ? y : 0;
    } else {
        static_assert(W == 64, "W must be 16, 32 or 64");
        return __builtin_amdgcn_update_dpp(0, x, 0x138, 0xF, 0xF, true);
    }
}

__device__ __forceinline__ int sat_sub(int x, int y) {
    // max(x - y, 0) for x >= 0, y >= 0
    return (int)__builtin_elementwise_sub_sat((unsigned)x, (unsigned)y);
}

__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }

// A gap cost as one 16-bit half of a packed operand.  Packed values never
// exceed 0x7BFF, so subtracting any cost of at least 0x7C00 saturates to 0,
// the same as subtracting the true cost: clamping at 0x7FFF keeps every
// result exact, while a cost of 65536 or more would otherwise be truncated
// and spill into the other pair's half.
__device__ __forceinline__ uint32_t cost16(int c) { return (uint32_t)(c < 0x7FFF ? c : 0x7FFF); }

struct PairJob {
    int64_t qbase, rbase;
    int n, m, dir, sid;
    int fwd_score, fwd_qe, fwd_re;
};

// The sub-problem of one pair for this sweep.  Pair ids come from the
// planning arrays; any id or length outside its documented range is an
// internal error, flagged and turned into an empty job.
// Extent of the reverse sweep of a pair whose forward pass found best score
// S > 0 ending at (qe, re): rows n = qe + 1 and columns m = re + 1 of the
// reversed prefixes, cut to the part that can hold a cell of score S.
// Every such cell (p, q) closes an alignment of score S that spans exactly p
// query and q reference residues (the forward end is the row-major-first
// maximum, so no S-scoring alignment from it ends earlier).  Such an
// alignment has at most min(p, q) aligned pairs, each scoring at most Mx,
// and at least |p - q| gap residues, which cost at least
// o + (k - 1) e for k of them when o >= e (k o when o < e).  So q - p is at
// most the largest k whose cost fits in Mx p - S, and likewise p - q.
// Cells right of or below the cut are never needed by those inside it, so
// the cut leaves every value inside, and the first S cell, unchanged.
__device__ __forceinline__ int gap_room(int64_t slack, int o, int e) {
    // largest number of gap residues whose least cost is at most `slack`
    if (o <= 0 || e < 0) return SW_MAX_REF;   // no bound
    if (slack < (int64_t)o) return 0;
    const int64_t k = o < e ? slack / o : (e == 0 ? (int64_t)SW_MAX_REF : 1 + (slack - o) / e);
    return k < (int64_t)SW_MAX_REF ? (int)k : SW_MAX_REF;
}
__device__ __forceinline__ void reverse_extent(int S, int Mx, int o, int e, int& n, int& m) {
    const int mq = n + gap_room((int64_t)Mx * n - S, o, e);
    if (m > mq) m = mq;
    const int np = m + gap_room((int64_t)Mx * m - S, o, e);
    if (n > np) n = np;
}

__device__ __forceinline__ PairJob load_job(const KParams& P, int pair, int reverse) {
    PairJob J;
    J.dir = 1; J.n = 0; J.m = 0; J.qbase = 0; J.rbase = 0; J.sid = 0;
    J.fwd_score = 0; J.fwd_qe = -1; J.fwd_re = -1;
    if (pair < 0) return J;
    if (pair >= *P.n_dev) {
        atomicOr(&P.flags[kFlagInternal], 1);
        return J;
    }
    J.sid = P.scheme_id ? (int)P.scheme_id[pair] : 0;
    const int64_t q0 = P.q_beg[pair], q1 = P.q_end[pair];
    const int64_t r0 = P.r_beg[pair], r1 = P.r_end[pair];
    if (!reverse) {
        J.qbase = q0; J.rbase = r0;
        J.n = (int)(q1 - q0); J.m = (int)(r1 - r0);
    } else {
        const sw_result f = P.out[pair];
        J.fwd_score = f.score; J.fwd_qe = f.q_end; J.fwd_re = f.r_end;
        if (f.score > 0) {
            J.n = f.q_end + 1; J.m = f.r_end + 1;
            J.qbase = q0 + f.q_end; J.rbase = r0 + f.r_end;
            J.dir = -1;
            if (J.sid < SW_MAX_SCHEMES)
                reverse_extent(f.score, P.max_score[J.sid], P.gap_open[J.sid], P.gap_extend[J.sid], J.n, J.m);
        }
    }
    if (J.n < 0 || J.n > SW_MAX_QUERY || J.m < 0 || J.m > SW_MAX_REF || J.sid >= SW_MAX_SCHEMES) {
        atomicOr(&P.flags[kFlagInternal], 1);
        J.n = 0; J.m = 0; J.sid = 0; J.fwd_score = 0;
    }
    return J;
}

// Drift group of column-word scheme sid.
__device__ __forceinline__ int drift_group(const KParams& P, int sid) { return (P.drift_of >> (8 * sid)) & 0xFF; }

// Leaves a pair of another drift group out of a sweep.  (Without a branch for the
// usual call of one group: it kept the loads of an item's pairs and of its
// residues apart, and 200,000 short DNA pairs were 1.3% slower.)
__device__ __forceinline__ void keep_group(const KParams& P, PairJob& J, int& pair) {
    const bool in = pair >= 0 && drift_group(P, J.sid) == P.group;
    J.n = in ? J.n : 0;
    J.m = in ? J.m : 0;
    J.fwd_score = in ? J.fwd_score : 0;
    pair = in ? pair : -1;
}

// Planning key of a pair of `bin` against m reference residues: the pairs of
// column-path schemes first, each part by decreasing length.  Drift groups follow
// one another in the first part, with coarser length buckets, so that few
// work items hold pairs of more than one.
__device__ __forceinline__ int pair_key(const KParams& P, int bin, bool col, int sid, int m) {
    const int b = kMHalf - 1 - m_bucket(m);
    if (!col) return bin * kMBuckets + kMHalf + b;
    const int shift = P.n_drift <= 1 ? 0 : P.n_drift == 2 ? 1 : 2;
    return bin * kMBuckets + drift_group(P, sid) * (kMHalf >> shift) + (b >> shift);
}

// Sets an error flag from any lanes (a plain store: every writer stores 1).
// No lane-divergent branch: see item_lane.
__device__ __forceinline__ void set_flag(int32_t* flags, int which, bool raise) {
    if (__builtin_amdgcn_ballot_w64(raise) != 0)
        __hip_atomic_store(&flags[which], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The lane index, taken from the hardware for each work item.  What must hold for
// the sweeps: this compiler has moved a register that stays live around a
// lane-divergent branch to another one inside the branch, where the lanes outside
// it keep their old contents, once registers were short.  So
//   * nothing is held per lane from one item to the next: the lane index and all
//     that is derived from it are made anew for every item (kept across items
//     they also fill registers that the sweep needs);
//   * within an item lane-divergent branches come only before its sweep (an
//     item's jobs: load_job, keep_group, box_job, trace_record), when only they and
//     the lane are live, and after it (results, push_redo), when only what they
//     write is; between, flags are raised by set_flag and residues are checked
//     without branches, and the rare branches of a sweep are taken by whole
//     wavefronts, on ballots.
__device__ __forceinline__ int item_lane() {
    int lane;
    asm volatile(
        "v_mbcnt_lo_u32_b32 %0, -1, 0\n\t"
        "v_mbcnt_hi_u32_b32 %0, -1, %0"
        : "=&v"(lane));
    return lane;
}

// Claims the next item of a queue: lane 0 adds 1 to its head and every lane
// gets the head's old value.  Written as one block with the execution mask
// set inside it: a lane-0 branch in the queue loop was once lowered into an
// inner loop that re-entered without the fetch, and an atomic of all lanes
// that adds 1 in lane 0 only became a loop over the 64 lanes.
__device__ __forceinline__ int next_item(int32_t* head) {
    int old;
    uint64_t saved;
    asm volatile(
        "s_mov_b64 %1, exec\n\t"
        "s_mov_b64 exec, 1\n\t"
        "global_atomic_add %0, %2, %3, off sc0\n\t"
        "s_waitcnt vmcnt(0)\n\t"
        "s_mov_b64 exec, %1"
        : "=&v"(old), "=&s"(saved)
        : "v"(head), "v"(1)
        : "memory");
    return __builtin_amdgcn_readfirstlane(old);
}

// Wave-scope ordering of LDS traffic: every lane's earlier LDS accesses are
// complete and visible before any lane's later ones (the wavefront executes
// in lock-step, so no workgroup barrier is needed).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Reference columns are streamed through LDS in chunks of C sweep steps
// (the tile width; kChunk unless a kernel is compiled for another).  While
// a chunk is swept, lanes read columns t0-W+1 .. t0+C+1 (the loop reads two
// steps ahead), so a group's buffer holds at least C+W+2 entries: entry x is
// column t0-W+x.  Each lane prefetches kPerLane entries of the next chunk
// into registers, so a narrower tile costs fewer registers and more chunk
// boundaries.  (kChunk and kChunkNarrow are in sw_internal.h.)

// A residue code of an alphabet of A, or `pad` outside the sequence and for
// an invalid code; `bad` becomes >= 0 when one inside it is invalid.
__device__ __forceinline__ int checked(int raw, bool inside, int A, int pad, int& bad) {
    const int x = inside ? raw : -1;
    bad = imax(bad, x - A);
    return (unsigned)x < (unsigned)A ? x : pad;
}

template <int W, int C = kChunk>
struct RefStager {
    static constexpr int kPerLane = (C + W + 2 + W - 1) / W;
    static constexpr int kBuf = kPerLane * W;
    int raw[kPerLane];

    // Issue the loads of the chunk starting at sweep step t0.  Addresses are
    // clamped into the pair's reference so that the loads are unconditional
    // and stay in flight while the previous chunk is swept.
    __device__ __forceinline__ void load(const uint8_t* refs, const PairJob& J, const void* dummy,
                                         int t0, int l) {
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) {
            int j = t0 - W + l + k * W;
            j = j < 0 ? 0 : (j >= J.m ? J.m - 1 : j);
            const uint8_t* p = J.m > 0 ? refs + J.rbase + (int64_t)J.dir * j
                                       : reinterpret_cast<const uint8_t*>(dummy);
            raw[k] = *p;
        }
    }
    // Write the chunk into the group's LDS buffer as matrix row offsets,
    // replacing out-of-range columns and invalid residues by the padding code.
    __device__ __forceinline__ void store(uint16_t* buf, const PairJob& J, int A, int t0, int l,
                                          int& bad) const {
        const int sbase = J.sid * kMatBytes;
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) {
            const int j = t0 - W + l + k * W;
            const int b = checked(raw[k], (unsigned)j < (unsigned)J.m, A, kPad, bad);
            buf[l + k * W] = (uint16_t)(sbase + b * kMatDim);
        }
    }
    // Pair-table path: write the chunk as byte offsets 2 b of the reference
    // residues into a pair-table row; out-of-range columns and invalid
    // residues get the padding code D - 1 (whose entries are 0, a score of -(o + e)).
    __device__ __forceinline__ void store_ptab(uint16_t* buf, const PairJob& J, int A, int D, int t0, int l,
                                               int& bad) const {
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) {
            const int j = t0 - W + l + k * W;
            const int b = checked(raw[k], (unsigned)j < (unsigned)J.m, A, D - 1, bad);
            buf[l + k * W] = (uint16_t)(2 * b);
        }
    }
    // Query-profile path: write the chunk as byte offsets b * row_bytes of
    // the reference residues' profile rows; out-of-range columns and invalid
    // residues get the padding code D - 1 (a row of zeros, a score of -(o + e)).
    __device__ __forceinline__ void store_qprof(uint16_t* buf, const PairJob& J, int A, int D, int row_bytes, int t0,
                                                int l, int& bad) const {
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) {
            const int j = t0 - W + l + k * W;
            const int b = checked(raw[k], (unsigned)j < (unsigned)J.m, A, D - 1, bad);
            buf[l + k * W] = (uint16_t)(row_bytes * b);
        }
    }
    // Small-alphabet path: write the chunk as column words (bytes M[a][b] + o + e
    // for a = 0..3); out-of-range columns and invalid residues get word 0
    // (the word of residue kPad, which no small alphabet holds).
    __device__ __forceinline__ void store_col(uint32_t* buf, const PairJob& J, int A, const uint32_t* colw,
                                              int t0, int l, int& bad) const {
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) {
            const int j = t0 - W + l + k * W;
            const int b = checked(raw[k], (unsigned)j < (unsigned)J.m, A, kPad, bad);
            buf[l + k * W] = colw[b];
        }
    }
};

// Per-block copy of the scoring schemes: substitution tables, column words
// of the small-alphabet path and gap costs.
struct SchemeLds {
    int8_t mat[SW_MAX_SCHEMES * kMatBytes];
    uint32_t colw[SW_MAX_SCHEMES][kMatDim];
    int32_t alphabet[SW_MAX_SCHEMES];
    int32_t gap_open[SW_MAX_SCHEMES];
    int32_t gap_extend[SW_MAX_SCHEMES];
    int32_t col_ok[SW_MAX_SCHEMES];
};

// Per-block copy for the pair-table sweep: the pair table of scheme
// P.ptab_sid (D^3 16-bit entries) and the gap costs of every scheme.
struct PtabLds {
    uint16_t tab[kPtabBytes / 2];
    uint8_t row_max[kMatDim];   // the scheme's best score of each query residue (0 for padding rows)
    int32_t alphabet[SW_MAX_SCHEMES];
    int32_t gap_open[SW_MAX_SCHEMES];
    int32_t gap_extend[SW_MAX_SCHEMES];
};

__device__ __forceinline__ void load_ptab(PtabLds& S, const KParams& P, int tid) {
    const int D = P.ptab_dim;
    const int words = (D > 0 && D <= kPtabMaxDim) ? (D * D * D + 1) / 2 : 0;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(P.mats + kPtabOffset);
    for (int k = tid; k < words; k += kBlock) reinterpret_cast<uint32_t*>(S.tab)[k] = src[k];
    if (tid < kMatDim) S.row_max[tid] = reinterpret_cast<const uint8_t*>(P.mats + kRowMaxOffset)[tid];
    if (tid < SW_MAX_SCHEMES) {
        S.alphabet[tid] = P.alphabet[tid];
        S.gap_open[tid] = P.gap_open[tid];
        S.gap_extend[tid] = P.gap_extend[tid];
    }
}

__device__ __forceinline__ void load_schemes(SchemeLds& S, const KParams& P, int tid) {
    for (int k = tid; k < SW_MAX_SCHEMES * kMatBytes / 4; k += kBlock)
        reinterpret_cast<int32_t*>(S.mat)[k] = reinterpret_cast<const int32_t*>(P.mats)[k];
    for (int k = tid; k < SW_MAX_SCHEMES * kMatDim; k += kBlock)
        (&S.colw[0][0])[k] = reinterpret_cast<const uint32_t*>(P.mats + SW_MAX_SCHEMES * kMatBytes)[k];
    if (tid < SW_MAX_SCHEMES) {
        S.col_ok[tid] = P.col_ok[tid];
        S.alphabet[tid] = P.alphabet[tid];
        S.gap_open[tid] = P.gap_open[tid];
        S.gap_extend[tid] = P.gap_extend[tid];
    }
}

// Counts the keys of a workgroup's pairs (PER per thread) in an LDS hash
// table and adds each distinct key's count to the global histogram at once,
// which also gives every pair its rank among the pairs of its key.  Bound by
// the global atomics: pairs of similar lengths share a few hundred keys in a
// few cache lines, where one atomic per pair, once to count and again to
// place, ran at 0.8 per ns (200,000 proteins against one query 260 + 260 us;
// now 20 + 5).  The table has twice as many slots as pairs, so a probe
// always ends.
template <int THREADS, int PER>
struct KeyCount {
    static constexpr int kLog = [] { int l = 1; while ((1 << l) < 2 * THREADS * PER) ++l; return l; }();
    static constexpr int kSlots = 1 << kLog;
    int32_t tag[kSlots], count[kSlots];
    __device__ __forceinline__ void clear() {
        for (int e = threadIdx.x; e < kSlots; e += THREADS) { tag[e] = -1; count[e] = 0; }
    }
    // (after a barrier) slot and rank within the workgroup; kTrivialKey is not counted
    __device__ __forceinline__ void insert(int key, int& slot, int& rank) {
        slot = rank = 0;
        if (key == kTrivialKey) return;
        int h = (int)(((uint32_t)key * 2654435761u) >> (32 - kLog));
        for (;;) {
            const int32_t was = atomicCAS(&tag[h], -1, key);
            if (was == -1 || was == key) break;
            h = (h + 1) & (kSlots - 1);
        }
        slot = h;
        rank = atomicAdd(&count[h], 1);
    }
    // (after a barrier) turn counts into the workgroup's first rank of each key
    __device__ __forceinline__ void reserve(int32_t* hist) {
        for (int e = threadIdx.x; e < kSlots; e += THREADS)
            if (count[e] > 0) count[e] = atomicAdd(&hist[tag[e]], count[e]);
    }
    // (after a barrier)
    __device__ __forceinline__ PairKey place(int key, int slot, int rank) const {
        PairKey k;
        k.key = key;
        k.rank = key == kTrivialKey ? 0 : count[slot] + rank;
        return k;
    }
};
// Calls of up to this many pairs are classified one pair per thread (enough
// workgroups for the device), larger ones 2048 pairs per workgroup, whose
// pairs share more keys.
constexpr int64_t kClassifySmall = 65536;

}  // namespace sw
