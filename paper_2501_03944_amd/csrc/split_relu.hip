// Fitness kernel instances: FP32 in two FP16 parts, weights staged in LDS, ReLU.
#include "fit_split.h"

namespace mgfwa {
namespace fit {

namespace {
// Eight wavefronts x 1 slab to a block, two such blocks on a compute unit where the
// weights leave the room, else the form with the most wavefronts whose accumulators (the
// cross products' beside the others) stay in registers.  512 sparks x 2,900 samples, best
// of 4 x 2 .. 16 x 1: 79 us at 32-64-10 (16 x 1 86), 93 at 32-96-10 (16 x 1 103), 123 at
// 32-128-10, 148 at 32-160-10 (16 x 1 153), 216 at 64-192-10 (12 x 1 242), 244 at
// 64-224-10, 276 at 64-256-10, 127 at 32-64-64-10 (8 x 2 140), 166 at 32-96-96-10 (16 x 1
// 178); 300 rows x 4,096 samples of 64-128-128-10 262 us (8 x 2 272).
const KernelEntry kEntries[] = {
    FIT_ENTRY_SPLIT(8, 1, 1, 4, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 1, 1, 6, 1, 0, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 8, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 2, 1, 10, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 1, 1, 12, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 1, 1, 14, 1, 0, 0),
    FIT_ENTRY_SPLIT(8, 1, 1, 16, 1, 0, 0),
    FIT_ENTRY_SPLIT(16, 1, 1, 4, 4, 1, 0),
    FIT_ENTRY_SPLIT(8, 2, 1, 4, 4, 1, 0),
    FIT_ENTRY_SPLIT(8, 1, 1, 6, 6, 1, 0),
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
