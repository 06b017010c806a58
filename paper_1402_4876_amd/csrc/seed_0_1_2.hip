// Seeded band kernel: score and end cell only, 32-bit scores, seed extension.
#include "seed.h"

namespace mica {
void reg_seed_0_1_2(KernelTable& t) {
  t.seed_band[0][1][2] = &k_seed_band<V32, 2, false>;
}
}  // namespace mica
