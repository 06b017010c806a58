// Seeded band kernel: score and end cell only, 32-bit scores, local.
#include "seed.h"

namespace mica {
void reg_seed_0_1_1(KernelTable& t) {
  t.seed_band[0][1][1] = &k_seed_band<V32, 1, false>;
}
}  // namespace mica
