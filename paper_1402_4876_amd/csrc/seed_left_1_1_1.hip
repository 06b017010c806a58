// Full traceback of the pairs the seeded band kernels leave: 32-bit scores,
// local, reads of more than 256 bases.
#include "seed.h"

namespace mica {
void reg_seed_left_1_1_1(KernelTable& t) { t.seed_left[1][1][1] = &k_seed_left<V32, 1, true>; }
}  // namespace mica
