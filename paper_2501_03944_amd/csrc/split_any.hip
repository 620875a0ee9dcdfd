// Fitness kernel instances: FP32 in two FP16 parts, weights staged in LDS, four layers
// in ReLU and two to four layers in any activation (chosen per layer at run time).
#include "fit_split.h"

namespace mgfwa {
namespace fit {

namespace {
const KernelEntry kEntries[] = {
    FIT_ENTRY_SPLIT(8, 1, 1, 4, 4, 4, 1),
    FIT_ENTRY_SPLIT(8, 2, 1, 6, 6, 6, 1),
    FIT_ENTRY_SPLIT(4, 1, -1, 4, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 1, -1, 8, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 1, -1, 16, 1, 0, 0),
    FIT_ENTRY_SPLIT(4, 1, -1, 4, 4, 1, 0),
    FIT_ENTRY_SPLIT(8, 1, -1, 8, 8, 1, 0),
    FIT_ENTRY_SPLIT(4, 1, -1, 4, 4, 4, 1),
};
}  // namespace

const KernelEntry *table_split_any(int *n)
{
    *n = (int)(sizeof kEntries / sizeof kEntries[0]);
    return kEntries;
}

}  // namespace fit
}  // namespace mgfwa
