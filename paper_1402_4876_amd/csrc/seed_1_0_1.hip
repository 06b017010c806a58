// Seeded band kernel: start and CIGAR, packed 16-bit scores, local.
#include "seed.h"

namespace mica {
void reg_seed_1_0_1(KernelTable& t) {
  t.seed_band[1][0][1] = &k_seed_band<V16, 1, true>;
}
}  // namespace mica
