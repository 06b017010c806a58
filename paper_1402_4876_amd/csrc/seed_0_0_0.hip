// Seeded band kernel: score and end cell only, packed 16-bit scores, semi-global (and the sample and scan of all modes).
#include "seed.h"

namespace mica {
void reg_seed_0_0_0(KernelTable& t) {
  t.seed_band[0][0][0] = &k_seed_band<V16, 0, false>;
  t.seed_sample[0][0] = &k_seed_sample<V16, false>;
  t.seed_scan[0][0] = &k_seed_scan<V16, false>;
}
}  // namespace mica
