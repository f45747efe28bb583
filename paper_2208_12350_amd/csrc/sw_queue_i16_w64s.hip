// sw_queue_i16_w64s.hip -- queue kernels of the packed int16 sweep shapes with
// 64-lane groups, 4, 6 and 8 rows per lane (queries up to 512 residues in
// small batches): table-lookup, column-word, pair-table and (forward only)
// query-profile kernels, forward and reverse.
#include "sw_queue.h"

namespace sw {

extern const KernelEntry kI16W64sKernels[];
extern const int kNumI16W64sKernels;

#define SW_ENTRY(W, R) \
    {16, W, R, {{{&sw_queue_kernel<16, W, R, false, false>, &sw_queue_kernel<16, W, R, true, false>}, \
                 {&sw_queue_kernel<16, W, R, false, true>, &sw_queue_kernel<16, W, R, true, true>}, \
                 {&sw_ptab_kernel<W, R, false>, &sw_ptab_kernel<W, R, true>}, \
                 {&sw_qprof_kernel<W, R>, nullptr}}, \
                {{nullptr, nullptr}, {nullptr, nullptr}, {nullptr, nullptr}, {nullptr, nullptr}}}},
const KernelEntry kI16W64sKernels[] = {
    SW_ENTRY(64, 4) SW_ENTRY(64, 6) SW_ENTRY(64, 8)
};
#undef SW_ENTRY
const int kNumI16W64sKernels = sizeof(kI16W64sKernels) / sizeof(kI16W64sKernels[0]);

// One launch per pass and score source serves every shape of this file.
extern const FamilyEntry kI16W64sFamily;
const FamilyEntry kI16W64sFamily = SW_FAMILY16(64, 2, 2, kChunk, 8, 6, 4);

}  // namespace sw
