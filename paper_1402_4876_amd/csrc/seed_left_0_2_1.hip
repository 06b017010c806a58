// Full traceback of the pairs the seeded band kernels leave: packed 16-bit scores,
// seed extension, reads of more than 256 bases.
#include "seed.h"

namespace mica {
void reg_seed_left_0_2_1(KernelTable& t) { t.seed_left[0][2][1] = &k_seed_left<V16, 2, true>; }
}  // namespace mica
