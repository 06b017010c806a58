// Size and memory of the interval table of the few-mismatch search.
//
// Plain C++, used by the index build (fm_build.hip) and built as host code by
// the CPU tests, which make its allocations fail one by one.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace mica {

// Bases of the table's strings: as many as keep it within twice the
// reference's length in bytes, 12 at most (134 MB).
constexpr int kFmMaxKmer = 12;
inline int fm_kmer_bases(uint64_t n) {
  int k = 0;
  while (k < kFmMaxKmer && (8ull << (2 * (k + 1))) <= 2 * n) ++k;
  return k;
}
// Bytes of the table, and of the level below it, which its construction needs
// beside it.
inline size_t fm_kmer_bytes(int k) { return (size_t)8 << (2 * k); }
inline size_t fm_kmer_tmp_bytes(int k) { return fm_kmer_bytes(k > 1 ? k - 1 : 1); }

// Memory of both: alloc(bytes) gives a pointer or NULL, release(p) takes it
// back.  The table is optional (a search without one steps through every base):
// without memory for either, both are NULL and nothing is held.
template <class Alloc, class Release>
bool fm_kmer_memory(int k, Alloc alloc, Release release, void** table, void** tmp) {
  *table = *tmp = nullptr;
  if (k < 1) return false;
  void* t = alloc(fm_kmer_bytes(k));
  if (!t) return false;
  void* u = alloc(fm_kmer_tmp_bytes(k));
  if (!u) {
    release(t);
    return false;
  }
  *table = t;
  *tmp = u;
  return true;
}

}  // namespace mica
