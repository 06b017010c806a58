// Seeded band kernel: start and CIGAR, 32-bit scores, local.
#include "seed.h"

namespace mica {
void reg_seed_1_1_1(KernelTable& t) {
  t.seed_band[1][1][1] = &k_seed_band<V32, 1, true>;
}
}  // namespace mica
