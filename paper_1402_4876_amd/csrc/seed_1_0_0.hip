// Seeded band kernel: start and CIGAR, packed 16-bit scores, semi-global (and the sample and scan of all modes).
#include "seed.h"

namespace mica {
void reg_seed_1_0_0(KernelTable& t) {
  t.seed_band[1][0][0] = &k_seed_band<V16, 0, true>;
  t.seed_sample[1][0] = &k_seed_sample<V16, true>;
  t.seed_scan[1][0] = &k_seed_scan<V16, true>;
}
}  // namespace mica
