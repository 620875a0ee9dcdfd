// Fitness kernel instances: FP32 in two FP16 parts, weights staged in LDS, ReLU.
#include "fit_split.h"

namespace mgfwa {
namespace fit {

namespace {
// 16 wavefronts x 1 slab where their registers allow it: 3-9 % ahead of 8 x 2 (one
// wavefront's conversions overlap the others' products), 512 sparks x 2,900 samples:
// 126 -> 114 us at 32-110-10, 198 -> 190 us at 64-192-10, 93 -> 87 us at 32-96-96-10.
const KernelEntry kEntries[] = {
    FIT_ENTRY_SPLIT(4, 4, 1, 4, 1, 0, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 6, 1, 0, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 8, 1, 0, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 10, 1, 0, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 12, 1, 0, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 14, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 2, 1, 16, 1, 0, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 16, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 2, 1, 4, 4, 1, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 6, 6, 1, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 8, 8, 1, 0),
    FIT_ENTRY_SPLIT(8, 2, 1, 8, 8, 1, 0),
    FIT_ENTRY_SPLIT(8, 2, 1, 10, 10, 1, 0),
};
}  // namespace

const KernelEntry *table_split(int *n)
{
    *n = (int)(sizeof kEntries / sizeof kEntries[0]);
    return kEntries;
}

}  // namespace fit
}  // namespace mgfwa
