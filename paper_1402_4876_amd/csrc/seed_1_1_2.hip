// Seeded band kernel: start and CIGAR, 32-bit scores, seed extension.
#include "seed.h"

namespace mica {
void reg_seed_1_1_2(KernelTable& t) {
  t.seed_band[1][1][2] = &k_seed_band<V32, 2, true>;
}
}  // namespace mica
