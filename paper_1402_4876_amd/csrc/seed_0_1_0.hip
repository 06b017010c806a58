// Seeded band kernel: score and end cell only, 32-bit scores, semi-global (and the sample and scan of all modes).
#include "seed.h"

namespace mica {
void reg_seed_0_1_0(KernelTable& t) {
  t.seed_band[0][1][0] = &k_seed_band<V32, 0, false>;
  t.seed_sample[0][1] = &k_seed_sample<V32, false>;
  t.seed_scan[0][1] = &k_seed_scan<V32, false>;
}
}  // namespace mica
