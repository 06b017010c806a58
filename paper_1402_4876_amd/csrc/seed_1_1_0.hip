// Seeded band kernel: start and CIGAR, 32-bit scores, semi-global (and the sample and scan of all modes).
#include "seed.h"

namespace mica {
void reg_seed_1_1_0(KernelTable& t) {
  t.seed_band[1][1][0] = &k_seed_band<V32, 0, true>;
  t.seed_sample[1][1] = &k_seed_sample<V32, true>;
  t.seed_scan[1][1] = &k_seed_scan<V32, true>;
}
}  // namespace mica
