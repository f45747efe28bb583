// sw_queue_i16_w256.hip -- queue kernels of the cooperative packed int16
// shapes (table-lookup, column-word and pair-table kernels): 256-lane groups (a workgroup's four wavefronts), 3..8 rows per
// lane (queries up to 2048 residues).
#include "sw_coop.h"

namespace sw {

extern const KernelEntry kI16W256Kernels[];
extern const int kNumI16W256Kernels;

#define SW_ENTRY(R) \
    {16, kCoopW, R, {{{&sw_coop_kernel<R, false, kVarTable>, &sw_coop_kernel<R, true, kVarTable>}, \
                      {&sw_coop_kernel<R, false, kVarCol>, &sw_coop_kernel<R, true, kVarCol>}, \
                      {&sw_coop_kernel<R, false, kVarPtab>, &sw_coop_kernel<R, true, kVarPtab>}, \
                      {nullptr, nullptr}}, \
                     {{nullptr, nullptr}, {nullptr, nullptr}, {nullptr, nullptr}, {nullptr, nullptr}}}},
const KernelEntry kI16W256Kernels[] = {
    SW_ENTRY(3) SW_ENTRY(4) SW_ENTRY(5) SW_ENTRY(6) SW_ENTRY(7) SW_ENTRY(8)
};
#undef SW_ENTRY
const int kNumI16W256Kernels = sizeof(kI16W256Kernels) / sizeof(kI16W256Kernels[0]);

// One launch per pass and score source serves every shape of this file.
extern const FamilyEntry kI16W256Family;
#define SW_COOP_FAMILY(VAR) {&sw_coop_family_kernel<false, VAR, 8, 7, 6, 5, 4, 3>, \
                             &sw_coop_family_kernel<true, VAR, 8, 7, 6, 5, 4, 3>}
const FamilyEntry kI16W256Family = {16, kCoopW, 6, {8, 7, 6, 5, 4, 3},
                                    {SW_COOP_FAMILY(kVarTable), SW_COOP_FAMILY(kVarCol), SW_COOP_FAMILY(kVarPtab)},
                                    {2, 2, 2}, {kChunk, kChunk, kChunk}};
#undef SW_COOP_FAMILY

}  // namespace sw
