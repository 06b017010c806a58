// Seeded band kernel: start and CIGAR, packed 16-bit scores, seed extension.
#include "seed.h"

namespace mica {
void reg_seed_1_0_2(KernelTable& t) {
  t.seed_band[1][0][2] = &k_seed_band<V16, 2, true>;
}
}  // namespace mica
