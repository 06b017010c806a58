// Full traceback of the pairs the seeded band kernels leave: 32-bit scores,
// semi-global, reads of up to 256 bases.
#include "seed.h"

namespace mica {
void reg_seed_left_1_0_0(KernelTable& t) { t.seed_left[1][0][0] = &k_seed_left<V32, 0, false>; }
}  // namespace mica
