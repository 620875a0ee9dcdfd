// Fitness kernel instances: weights staged in LDS, two to four layers in any activation
// (chosen per layer at run time), and four layers in ReLU, in FP32 and BF16.  From global
// memory, rows that are not aligned are read value by value for every slab (17-40-33-20-3,
// 2,500 rows x 1,029 samples: 1,282 us, so 829 us) and wide ones overflow the registers
// (112 sparks x 6,013 samples of 32-103-103-103-10: 1,020 us, so 377 us); 1,200
// sparks x 1,067 samples of 30-71-71-2 in BF16 1,400 -> 811 us a generation.
#include "fit_kernel.h"

namespace mgfwa {
namespace fit {

namespace {
const KernelEntry kEntries[] = {
    FIT_ENTRY_SCHED(false, true, 4, 2, -1, 5, 8, 1, 0, 0),
    FIT_ENTRY_SCHED(true, true, 4, 2, -1, 5, 8, 1, 0, 0),
    FIT_ENTRY_SCHED(false, true, 4, 2, -1, 5, 16, 1, 0, 0),
    FIT_ENTRY_SCHED(true, true, 4, 2, -1, 5, 16, 1, 0, 0),
    FIT_ENTRY_SCHED(false, true, 4, 2, -1, 5, 4, 4, 1, 0),
    FIT_ENTRY_SCHED(true, true, 4, 2, -1, 5, 4, 4, 1, 0),
    FIT_ENTRY_SCHED(false, true, 4, 2, -1, 5, 8, 8, 1, 0),
    FIT_ENTRY_SCHED(true, true, 4, 2, -1, 5, 8, 8, 1, 0),
    FIT_ENTRY_SCHED(false, true, 4, 2, -1, 5, 4, 4, 4, 1),
    FIT_ENTRY_SCHED(true, true, 4, 2, -1, 5, 4, 4, 4, 1),
    FIT_ENTRY_SCHED(true, true, 4, 4, 1, 7, 2, 2, 2, 1),
    FIT_ENTRY_SCHED(true, true, 4, 2, 1, 7, 4, 4, 4, 1),
    FIT_ENTRY_SCHED(true, true, 8, 2, 1, 7, 8, 8, 8, 1),
    FIT_ENTRY_SCHED(false, true, 4, 4, 1, 5, 2, 2, 2, 1),
    FIT_ENTRY_SCHED(false, true, 4, 2, 1, 5, 4, 4, 4, 1),
    FIT_ENTRY_SCHED(false, true, 16, 1, 1, 5, 7, 7, 7, 1),
    FIT_ENTRY_SCHED(false, true, 4, 2, -1, 5, 7, 7, 7, 1),
};
}  // namespace

const KernelEntry *table_lds_any(int *n)
{
    *n = (int)(sizeof kEntries / sizeof kEntries[0]);
    return kEntries;
}

}  // namespace fit
}  // namespace mgfwa
