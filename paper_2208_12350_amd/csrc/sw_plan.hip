// sw_plan.hip -- device-side planning of a sweep pass (gfx950).
//
// For each pass (forward, then reverse) the pairs are
//   1. classified: validated (forward), routed to int16 or int32 by their
//      score bound, given a bin from their (sub)query length and a 16-bit
//      key (bin, reference-length bucket, longest first);
//   2. counted into a histogram of keys, which also gives each pair its rank
//      among the pairs of its key (KeyCount);
//   3. the histogram is scanned into bucket offsets and per-bin pair and
//      work-item ranges, one workgroup per bin;
//   4. pairs move to their offset plus rank, in key order (order within a
//      bucket is irrelevant: every pair's result is independent of where it
//      runs), and are cut into wavefront work items of ppw consecutive pairs
//      of one bin.
// That is three launches: in small calls each costs about 10 us, more than
// its work.
// The reverse pass re-bins pairs by the shape of their reverse sub-problem
// (q_end+1 rows, r_end+1 columns), which can differ a lot from the forward
// shape.  Nothing here synchronises with the host and nothing is cleared
// with a memset, so a whole call can be captured in a hipGraph.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sw_device.h"
#include "sw_internal.h"

namespace sw {

__global__ void sw_reset_kernel(int32_t* p, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

__global__ void sw_call_start_kernel(int32_t* small, int n_small, int32_t* hist, int n_hist, int32_t* n_dev,
                                     int32_t n_pairs) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_hist; i += gridDim.x * blockDim.x) {
        hist[i] = 0;
        if (i < n_small) small[i] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_dev = n_pairs;
}

template <int THREADS, int PER>
__global__ __launch_bounds__(THREADS) void sw_classify_kernel(KParams P, ClassifyArgs C, const int8_t* lut,
                                                              const BinInfo* bins, PairKey* keys, int32_t* hist,
                                                              unsigned long long* counters) {
    const int64_t n_pairs = *P.n_dev;
    // counters[0] / [1]: forward / reverse cells; counters[2]: int32 pairs
    // (forward); per bin of this pass: cells and pairs (kCtrBinCells,
    // kCtrBinPairs, indexed pass * kMaxBins + bin)
    __shared__ KeyCount<THREADS, PER> KC;
    __shared__ unsigned long long s_cells;
    __shared__ int32_t s_i32;
    __shared__ unsigned long long s_bin_cells[2][kMaxBins];   // [column path?][bin]
    __shared__ uint32_t s_bin_pairs[2][kMaxBins];
    KC.clear();
    if (threadIdx.x == 0) { s_cells = 0; s_i32 = 0; }
    if (threadIdx.x < kMaxBins) {
        s_bin_cells[0][threadIdx.x] = s_bin_cells[1][threadIdx.x] = 0;
        s_bin_pairs[0][threadIdx.x] = s_bin_pairs[1][threadIdx.x] = 0;
    }
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * (THREADS * PER) + threadIdx.x;
    int key[PER], slot[PER], rank[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t i = i0 + u * THREADS;
        key[u] = kTrivialKey;
        if (i < n_pairs) {
            int64_t n = 0, m = 0;
            int s = 0;
            bool ok = false;
            if (!P.reverse) {
                n = P.q_end[i] - P.q_beg[i];
                m = P.r_end[i] - P.r_beg[i];
                s = P.scheme_id ? (int)P.scheme_id[i] : 0;
                if (n < 0 || m < 0) atomicOr(&P.flags[kFlagBadOffsets], 1);
                else if (s >= C.n_schemes) atomicOr(&P.flags[kFlagBadScheme], 1);
                else if (n > SW_MAX_QUERY || m > SW_MAX_REF || (C.max_query > 0 && n > C.max_query))
                    atomicOr(&P.flags[kFlagTooLong], 1);
                else ok = n > 0 && m > 0;
                if (!ok) {
                    sw_result z;
                    z.score = 0; z.q_start = z.q_end = z.r_start = z.r_end = -1;
                    P.out[i] = z;
                }
            } else {
                // the reverse sub-problem is the prefix box ending at the forward
                // end; an end outside the pair would be an internal error
                const sw_result r = P.out[i];
                if (r.score > 0) {
                    const int64_t n0 = P.q_end[i] - P.q_beg[i];
                    const int64_t m0 = P.r_end[i] - P.r_beg[i];
                    n = (int64_t)r.q_end + 1;
                    m = (int64_t)r.r_end + 1;
                    s = P.scheme_id ? (int)P.scheme_id[i] : 0;
                    ok = n >= 1 && n <= n0 && m >= 1 && m <= m0 && s < C.n_schemes;
                    if (!ok) {
                        atomicOr(&P.flags[kFlagInternal], 1);
                    } else {
                        // the part of the prefixes that can hold the start (the
                        // sweep cuts its job the same way)
                        int nn = (int)n, mm = (int)m;
                        reverse_extent(r.score, P.max_score[s], P.gap_open[s], P.gap_extend[s], nn, mm);
                        n = nn;
                        m = mm;
                    }
                }
            }
            if (ok) {
                const int64_t mn = n < m ? n : m;
                const int sel = (mn * C.max_score[s] <= C.i16_limit && m <= kI16MaxRef) ? 0 : 1;
                if (sel && !P.reverse) atomicAdd(&s_i32, 1);
                const int lut_sel = sel ? kLutI32 : C.col_ok[s] ? kLutI16Col : kLutI16;
                const int bin = lut[lut_sel * kLutRows + (int)((n - 1) / 16)];
                // within a bin: pairs of column-path schemes first (the bin's
                // column-word kernel takes them), each part by decreasing
                // reference length; only packed-int16 pairs use column words
                const int col = (sel == 0 && C.col_ok[s] && bins[bin].col) ? 1 : 0;
                key[u] = pair_key(P, bin, col != 0, s, (int)m);
                atomicAdd(&s_bin_cells[col][bin], (unsigned long long)(n * m));
                atomicAdd(&s_bin_pairs[col][bin], 1u);
            }
        }
        KC.insert(key[u], slot[u], rank[u]);
    }
    __syncthreads();
    KC.reserve(hist);
    if (threadIdx.x < kMaxBins) {
        const unsigned long long cells = s_bin_cells[0][threadIdx.x] + s_bin_cells[1][threadIdx.x];
        if (cells) atomicAdd(&s_cells, cells);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t i = i0 + u * THREADS;
        if (i < n_pairs) keys[i] = KC.place(key[u], slot[u], rank[u]);
    }
    if (threadIdx.x == 0) {
        if (s_cells) atomicAdd(&counters[P.reverse ? kCtrRevCells : kCtrFwdCells], s_cells);
        if (s_i32) atomicAdd(&counters[kCtrI32Pairs], (unsigned long long)s_i32);
    }
    if (threadIdx.x < kMaxBins) {
        const int b = threadIdx.x;
        const int slot = (P.reverse ? kMaxBins : 0) + b;
        const unsigned long long pairs = s_bin_pairs[0][b] + s_bin_pairs[1][b];
        if (pairs) {
            atomicAdd(&hist[kHistPairs + b], (int32_t)pairs);
            atomicAdd(&counters[kCtrBinCells + slot], s_bin_cells[0][b] + s_bin_cells[1][b]);
            atomicAdd(&counters[kCtrBinPairs + slot], pairs);
        }
        if (s_bin_pairs[1][b]) {
            atomicAdd(&hist[kHistCol + b], (int32_t)s_bin_pairs[1][b]);
            atomicAdd(&counters[kCtrBinColCells + slot], s_bin_cells[1][b]);
            atomicAdd(&counters[kCtrBinColPairs + slot], (unsigned long long)s_bin_pairs[1][b]);
        }
    }
}

// Inclusive scan within a wavefront.
__device__ __forceinline__ int32_t wave_scan(int32_t v, int lane) {
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t u = __shfl_up(v, off);
        if (lane >= off) v += u;
    }
    return v;
}

// Plan of a pass from the classified pairs' histogram, whose last entries
// are every bin's pairs and column-path pairs.  Workgroup b < kMaxBins scans
// bin b's kMBuckets entries in place, offset by the pairs of bins 0..b-1;
// workgroup kMaxBins writes the metadata.  The column-path pairs (the first half of a
// bin's keys) and the others are cut into items separately, so no item mixes
// the two.  Bound by the latency of its loads: the ranges of all bins come
// from one scan over the lanes (21 us with a loop over the bins, now 6).
constexpr int kBinScanThreads = 256;
constexpr int kBinScanRun = kMBuckets / kBinScanThreads;
static_assert(kMaxBins <= 128, "bin ranges are scanned by two wavefronts");

__global__ __launch_bounds__(kBinScanThreads) void sw_plan_bins_kernel(const BinInfo* bins, int n_bins,
                                                                        int32_t* hist, int32_t* meta) {
    __shared__ int32_t s_tot[2], s_base;
    __shared__ int32_t wave_tot[kBinScanThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int b = blockIdx.x;
    // the first two wavefronts: thread t has bin t
    const bool real = t < kMaxBins && t < n_bins;
    const int32_t pairs = real ? hist[kHistPairs + t] : 0;
    int32_t v[kBinScanRun];
    int32_t* hb = hist + b * kMBuckets + t * kBinScanRun;
    if (b < kMaxBins) {
#pragma unroll
        for (int k = 0; k < kBinScanRun; ++k) v[k] = hb[k];
    }
    const int32_t pos = wave_scan(pairs, lane) - pairs;
    if (lane == 63 && wave < 2) s_tot[wave] = pos + pairs;
    __syncthreads();
    const int32_t first = pos + (wave == 1 ? s_tot[0] : 0);   // of bin t
    if (b < kMaxBins) {
        int32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kBinScanRun; ++k) sum += v[k];
        const int32_t incl = wave_scan(sum, lane);
        if (lane == 63) wave_tot[wave] = incl;
        if (t == b) s_base = first;
        __syncthreads();
        int32_t run = s_base + incl - sum;
        for (int w = 0; w < wave; ++w) run += wave_tot[w];
#pragma unroll
        for (int k = 0; k < kBinScanRun; ++k) {
            hb[k] = run;
            run += v[k];
        }
        return;
    }
    const int32_t col = real && bins[t].col ? hist[kHistCol + t] : 0;
    const int32_t ppw = real ? bins[t].ppw : 1;
    const int32_t col_items = (col + ppw - 1) / ppw;
    const int32_t items = col_items + (pairs - col + ppw - 1) / ppw;
    const int32_t ipos = wave_scan(items, lane) - items;
    __syncthreads();
    const int32_t total = s_tot[0] + s_tot[1];
    __syncthreads();
    if (lane == 63 && wave < 2) s_tot[wave] = ipos + items;
    __syncthreads();
    if (t < kMaxBins) {
        const int32_t ifirst = ipos + (wave == 1 ? s_tot[0] : 0);
        meta[kMetaBinFirst + t] = first;
        meta[kMetaItemFirst + t] = ifirst;
        meta[kMetaItemSplit + t] = ifirst + col_items;
        meta[kMetaBinCol + t] = col;
        meta[kMetaHeads + t] = 0;
        for (int g = 0; g < SW_MAX_SCHEMES; ++g) meta[kMetaColHeads + g * kMaxBins + t] = 0;
    }
    if (t == 0) {
        meta[kMetaBinFirst + kMaxBins] = total;
        meta[kMetaItemFirst + kMaxBins] = s_tot[0] + s_tot[1];
        meta[kMetaRedo] = 0;
    }
}

// Thread i moves pair i to its sorted position and, for sorted position i,
// writes the work item that begins there (which depends on the ranges only).
// Pairs with the trivial key get no position: nothing reads the sorted order
// past the last bin (their results, if any, were written at classification).
__global__ void sw_scatter_kernel(const PairKey* keys, const int32_t* meta, const BinInfo* bins, int n_bins,
                                  const int32_t* n_dev, const int32_t* offs, int32_t* order, WorkItem* items) {
    __shared__ int32_t s_first[kMaxBins + 1];
    if (threadIdx.x <= kMaxBins) s_first[threadIdx.x] = meta[kMetaBinFirst + threadIdx.x];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= *n_dev) return;
    const PairKey pk = keys[i];
    if (pk.key != kTrivialKey) order[offs[pk.key] + pk.rank] = (int32_t)i;
    if (i >= s_first[n_bins]) return;
    // the bin holding sorted position i: the last bin whose first position
    // is at most i (empty bins share their successor's first position)
    int lo = 0, hi = n_bins - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_first[mid] <= i) lo = mid;
        else hi = mid - 1;
    }
    const int b = lo;
    const int32_t f = s_first[b];
    const int32_t cnt = s_first[b + 1] - f;
    const int32_t ncol = meta[kMetaBinCol + b];
    const BinInfo bi = bins[b];
    // column-path pairs [0, ncol) of the bin, then the others, each cut
    // into items of ppw pairs
    int32_t k = (int32_t)i - f, end = ncol, item = meta[kMetaItemFirst + b];
    if (k >= ncol) {
        k -= ncol;
        end = cnt - ncol;
        item += (ncol + bi.ppw - 1) / bi.ppw;
    }
    if (k % bi.ppw != 0) return;
    WorkItem w;
    w.first = (int32_t)i;
    w.count = (uint16_t)(end - k < bi.ppw ? end - k : bi.ppw);
    w.bin = (uint8_t)b;
    w.pad = 0;
    items[item + k / bi.ppw] = w;
}

__global__ void sw_fill_span_kernel(int64_t* beg, int64_t* end, int64_t n, int64_t len) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        beg[i] = 0;
        end[i] = len;
    }
}

static unsigned grid_for(int64_t n, int threads) {
    int64_t b = (n + threads - 1) / threads;
    return (unsigned)(b > 0 ? b : 1);
}

hipError_t launch_fill_span(int64_t* beg, int64_t* end, int64_t n, int64_t len, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    unsigned blocks = grid_for(n, 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(sw_fill_span_kernel, dim3(blocks), dim3(256), 0, s, beg, end, n, len);
    return hipGetLastError();
}

hipError_t launch_reset(int32_t* p, int n, hipStream_t s) {
    unsigned blocks = grid_for(n, 256);
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(sw_reset_kernel, dim3(blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_call_start(int32_t* small, int n_small, int32_t* hist, int n_hist, int32_t* n_dev, int32_t n_pairs,
                             hipStream_t s) {
    unsigned blocks = grid_for(n_hist, 1024);
    hipLaunchKernelGGL(sw_call_start_kernel, dim3(blocks), dim3(256), 0, s, small, n_small, hist, n_hist, n_dev,
                       n_pairs);
    return hipGetLastError();
}

hipError_t launch_classify(const KParams& P, const ClassifyArgs& C, const int8_t* lut, const BinInfo* bins,
                           int64_t cap, PairKey* keys, int32_t* hist,
                           unsigned long long* counters, hipStream_t s) {
    if (cap <= 0) return hipSuccess;
    if (cap <= kClassifySmall)
        hipLaunchKernelGGL((sw_classify_kernel<256, 1>), dim3(grid_for(cap, 256)), dim3(256), 0, s, P, C, lut, bins,
                           keys, hist, counters);
    else
        hipLaunchKernelGGL((sw_classify_kernel<1024, 2>), dim3(grid_for(cap, 2048)), dim3(1024), 0, s, P, C, lut,
                           bins, keys, hist, counters);
    return hipGetLastError();
}

hipError_t launch_plan_bins(const BinInfo* bins, int n_bins, int32_t* hist, int32_t* meta, hipStream_t s) {
    hipLaunchKernelGGL(sw_plan_bins_kernel, dim3(kMaxBins + 1), dim3(kBinScanThreads), 0, s, bins, n_bins, hist,
                       meta);
    return hipGetLastError();
}

hipError_t launch_scatter(const PairKey* keys, const int32_t* meta, const BinInfo* bins, int n_bins,
                          const int32_t* n_dev, int64_t cap, const int32_t* hist, int32_t* order, WorkItem* items,
                          hipStream_t s) {
    if (cap <= 0) return hipSuccess;
    hipLaunchKernelGGL(sw_scatter_kernel, dim3(grid_for(cap, 256)), dim3(256), 0, s, keys, meta, bins, n_bins, n_dev,
                       hist, order, items);
    return hipGetLastError();
}

}  // namespace sw
