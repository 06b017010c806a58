// Seeded band kernel: score and end cell only, packed 16-bit scores, local.
#include "seed.h"

namespace mica {
void reg_seed_0_0_1(KernelTable& t) {
  t.seed_band[0][0][1] = &k_seed_band<V16, 1, false>;
}
}  // namespace mica
