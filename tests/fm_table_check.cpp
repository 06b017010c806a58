// The interval table's memory (paper_1402_4876_amd/csrc/fm_table.h) as host
// code under AddressSanitizer (tests/test_fm_table_memory.py): with every
// allocation, with the first and with the second failing, at every size of the
// table's strings.  A failure gives back what was held and means no table.
// Exit status 0 = no sanitizer report and every check passed.
#include <cstdio>
#include <cstdlib>
#include <set>

#include "fm_table.h"

using namespace mica;

int main() {
  int failures = 0;
  auto check = [&](bool ok, const char* what, int k) {
    if (!ok) {
      std::printf("k %d: %s\n", k, what);
      ++failures;
    }
  };
  for (uint64_t n = 1; n < 1u << 28; n = n * 3 / 2 + 1) {
    const int k = fm_kmer_bases(n);
    check(k == 0 || fm_kmer_bytes(k) <= 2 * n, "table past twice the reference", k);
    check(k == kFmMaxKmer || fm_kmer_bytes(k + 1) > 2 * n, "table could be larger", k);
  }
  for (int k = 0; k <= kFmMaxKmer; ++k) {
    // the construction writes levels 1..k in turn, the last one to the table
    for (int level = k - 1; level >= 1; level -= 2)
      check(fm_kmer_bytes(level) <= fm_kmer_tmp_bytes(k), "temporary level too large", k);
    for (int fails = 0; fails < 3; ++fails) {  // the allocation that fails, 0: none
      std::set<void*> held;
      int calls = 0;
      auto alloc = [&](size_t bytes) -> void* {
        if (++calls == fails) return nullptr;
        void* p = std::malloc(bytes);
        held.insert(p);
        return p;
      };
      auto release = [&](void* p) {
        check(held.erase(p) == 1, "released what it does not hold", k);
        std::free(p);
      };
      void *table = &failures, *tmp = &failures;
      const bool got = fm_kmer_memory(k, alloc, release, &table, &tmp);
      check(got == (k > 0 && fails == 0), "table with a failed allocation, or none without", k);
      check(got ? table && tmp && held.size() == 2 : !table && !tmp && held.empty(), "memory kept", k);
      if (got) {
        release(table);
        release(tmp);
      }
    }
  }
  std::printf(failures ? "%d failures\n" : "table memory ok\n", failures);
  return failures ? 1 : 0;
}
