// Full traceback of the pairs the seeded band kernels leave: 32-bit scores,
// seed extension, reads of up to 256 bases.
#include "seed.h"

namespace mica {
void reg_seed_left_1_2_0(KernelTable& t) { t.seed_left[1][2][0] = &k_seed_left<V32, 2, false>; }
}  // namespace mica
