// sw_queue_i32_all.hip -- one kernel for every int32 shape: what a pass
// launches for the few pairs, most often none, that do not fit the packed
// int16 sweeps.  (In a file of its own: beside the kernels of single shapes
// the compiler allocates those differently, 7% slower.)
#include "sw_queue.h"

namespace sw {

template <bool REV, int... R64, int... R16>
__device__ __forceinline__ void members32(const KParams& P, SchemeLds& L, uint16_t* wbuf, int lane, int n_pairs,
                                          std::integer_sequence<int, R64...>, std::integer_sequence<int, R16...>) {
    int k = 0;
    ((family_member<32, 64, R64, REV, kVarTable, kChunk, SchemeLds>(P, L, wbuf, lane, P.fam_bins[k++], n_pairs)), ...);
    ((family_member<32, 16, R16, REV, kVarTable, kChunk, SchemeLds>(P, L, wbuf, lane, P.fam_bins[k++], n_pairs)), ...);
}
template <bool REV>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) void sw_family32_kernel(KParams P) {
    __shared__ __attribute__((aligned(16))) SchemeLds L;
    __shared__ uint16_t wbufs[kWavesPerBlock * kWaveBuf];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int items = 0;
    for (int m = 0; m < kFamilyMax; ++m) {
        const int bin = P.fam_bins[m];
        if (bin >= 0) items += P.meta[kMetaItemFirst + bin + 1] - P.meta[kMetaItemSplit + bin];
    }
    if (__builtin_amdgcn_readfirstlane(items) == 0) return;
    load_schemes(L, P, tid);
    const int n_pairs = __builtin_amdgcn_readfirstlane(*P.n_dev);
    __syncthreads();
    members32<REV>(P, L, wbufs + wave * kWaveBuf, lane, n_pairs,
                   std::integer_sequence<int, 32, 28, 24, 20, 16, 14, 12, 10, 8, 6>{},
                   std::integer_sequence<int, 16, 14, 12, 10, 8, 6, 4, 2>{});
}
extern const FamilyEntry kI32Family;
const FamilyEntry kI32Family = {32, 0, 18, {32, 28, 24, 20, 16, 14, 12, 10, 8, 6, 16, 14, 12, 10, 8, 6, 4, 2},
                                       {{&sw_family32_kernel<false>, &sw_family32_kernel<true>},
                                        {nullptr, nullptr}, {nullptr, nullptr}},
                                       {2, 2, 2}, {kChunk, kChunk, kChunk},
                                       {64, 64, 64, 64, 64, 64, 64, 64, 64, 64, 16, 16, 16, 16, 16, 16, 16, 16}};

}  // namespace sw
