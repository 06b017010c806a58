// Seeded band kernel: score and end cell only, packed 16-bit scores, seed extension.
#include "seed.h"

namespace mica {
void reg_seed_0_0_2(KernelTable& t) {
  t.seed_band[0][0][2] = &k_seed_band<V16, 2, false>;
}
}  // namespace mica
