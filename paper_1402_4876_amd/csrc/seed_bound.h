// What a loss proves about an alignment (the bounds of the seeded band
// kernels; seed.h says how they are used).
//
// Plain integer code, used by the kernels and the host runtime and built as
// host C++ by the CPU tests (which define the __host__ / __device__ /
// __forceinline__ keywords away), where the bounds are held against full
// tables under random scorings.
//
// Let a be the match score and call a m - score the loss of an alignment of a
// read of m bases: a - b per substitution, o + L e per deletion run, o + L (a
// + e) per insertion run, a per clipped base.  The read is cut into T = m /
// kSeed parts of kSeed bases.  A part that the alignment does not match
// exactly along one diagonal is spoiled, and every spoiled part lies under
// some event:
// - a substitution spoils one part, a deletion run at most one;
// - an insertion run of L bases touches one part (L = 1) or at most 2 +
//   (L - 2) / kSeed: it has to swallow kSeed bases for each part past the
//   second;
// - a clipped end spoils the first or the last part with its first bases,
//   each further part with kSeed of them, kSeed a each.
// So k spoiled parts cost at least k c, c the least of these per part
// (spoil_cost2), where in local mode the first and the last part may be
// spoiled for nothing.
//
// Losses are doubled throughout: the open of a split run is shared by two
// parts.
#pragma once
#include <stdint.h>

namespace mica {

constexpr int kSeed = 12;  // bases of a read part: 24 bits, and 8 for its number

// The scoring, and twice the least loss per spoiled part: of any alignment, of
// a stretch beside the gap that leads there, and beside a run that moves the
// alignment (which may be split).
struct SeedCosts {
  int a, open, ext;
  int cost2, cost2_local;
  int leave2, leave2_local;
  int move2_del, move2_ins;
  // 2^32 over twice e, a + e and a + 2 e, rounded up
  uint32_t per_del, per_ins, per_both;
};

// Twice the least loss per spoiled part: a substitution or a deletion spoils
// one; an insertion run that touches s parts has L >= 1, 2, 2 + (s - 2) kSeed,
// ... bases and costs o + L (a + e) for the s.
inline int spoil_cost2(int a, int b, int o, int e, int max_parts) {
  int c2 = 2 * (a - b < o + e ? a - b : o + e);
  for (int k = 1; k <= max_parts; ++k) {
    const int len = k <= 2 ? k : 2 + (k - 2) * kSeed;
    const int v = 2 * (o + len * (a + e)) / k;
    c2 = v < c2 ? v : c2;
  }
  return c2;
}

inline SeedCosts seed_costs(int a, int b, int o, int e, int max_parts) {
  auto least = [](int x, int y) { return x < y ? x : y; };
  SeedCosts c;
  c.a = a;
  c.open = o;
  c.ext = e;
  c.cost2 = spoil_cost2(a, b, o, e, max_parts);
  c.cost2_local = least(c.cost2, 2 * kSeed * a);
  // off the diagonal, next to the gap that led there: an inserted run may have
  // spoiled whole parts, each with its kSeed bases
  c.leave2 = least(c.cost2, 2 * kSeed * (a + e));
  c.leave2_local = least(c.cost2_local, c.leave2);
  // beside a run: splitting it costs o for each part saved (two for
  // insertions); a clipped end spoils its further parts with kSeed bases each
  const int move2 = least(c.leave2, 2 * kSeed * a);
  c.move2_del = least(move2, 2 * o);
  c.move2_ins = least(move2, o);
  auto over = [](int per) { return (uint32_t)(((1ull << 32) + 2 * (uint64_t)per - 1) / (2 * (uint64_t)per)); };
  c.per_del = over(e);
  c.per_ins = over(a + e);
  c.per_both = over(a + 2 * e);
  return c;
}

// The core of a pair: the span of the diagonals of its parts' occurrences; the
// fewer occurrences of the two when they are exactly two diagonals (else 0);
// the parts without occurrence.  In local mode the first and the last part, which
// clipping spoils for nothing, count in neither.
struct Core {
  int span, hmin, missed;
};
__host__ __device__ __forceinline__ uint32_t core_word(const Core& c) {
  return (uint32_t)c.span | ((uint32_t)c.hmin << 8) | ((uint32_t)c.missed << 16);
}
__host__ __device__ __forceinline__ Core core_of(uint32_t w) {
  return Core{(int)(w & 0xFFu), (int)((w >> 8) & 0xFFu), (int)(w >> 16)};
}

// The certificate of T parts: an alignment of this loss matches one exactly.
__host__ __device__ __forceinline__ bool loss_certain(const SeedCosts& c, bool local, int T, int loss) {
  const int parts = local ? T - 2 : T;
  return parts > 0 && 2 * loss < parts * (local ? c.cost2_local : c.cost2);
}

// The parts that w inserted bases swallow past the two that each run touches.
__host__ __device__ __forceinline__ int swallowed(int w) { return w > 2 ? (w - 2) / kSeed : 0; }

// The bases that a doubled loss left2 pays for, 2^32 / per their doubled price
// rounded up (so the quotient is never too low; a division takes some 20
// instructions).
__host__ __device__ __forceinline__ int paid_bases(int left2, uint32_t per) {
  return left2 > 0 ? (int)(((uint64_t)(uint32_t)left2 * per) >> 32) : 0;
}

// The most inserted bases that left2 pays for beside `parts` parts of cost2
// each, of which the bases swallow some.  (Not monotone: a base that completes a
// part may pay for itself.  Every allowed number is at most what the parts it
// leaves allow, so it stays at most w as w falls from what no part at all allows
// to the largest number that holds.)
__host__ __device__ __forceinline__ int inserted_bases(int left2, uint32_t per, int parts, int cost2) {
  int w = paid_bases(left2, per), k;
  if (parts <= 0) return w;
  do {
    k = swallowed(w);
    w = paid_bases(left2 - (parts > k ? (parts - k) * cost2 : 0), per);
  } while (swallowed(w) != k);
  return w;
}

// Diagonals an alignment of loss `loss`, which matches a part exactly, can
// move off the core (bounds from above).
//
// It spoils the parts without occurrence and, if it matches no part of one of
// two diagonals, the hmin parts there, P in all.  Moving w diagonals takes w
// deleted or w inserted bases:
//   deletions     o + w e       + (P - 1) cd
//   insertions    o + w (a + e) + (P - 2 - swallowed(w)) ci
// as a run touches one part (two), each further run costs o for one part
// more (two) and every other event c for each part: cd = min(c, o), ci = min(c,
// o / 2).
//
// If it matches parts on both diagonals, span s apart, P is only the parts
// without occurrence, but there are two runs at least, and by the order in
// which it visits the two diagonals and the one w past them, it deletes s + w
// bases (in two runs, or beside w or s inserted ones) or inserts s + w:
//   2 o + (s + w) e               + (P - 2) cd
//   2 o + (s + w) e + w (a + e)   + (P - 3 - swallowed(w)) ci
//   2 o + (s + w) e + i (a + e)   + (P - 3 - swallowed(i)) ci,  i >= s
//   2 o + (s + w) (a + e)         + (P - 4 - swallowed(s + w)) ci
// In the third the parts that a longer i swallows cost no less than their
// bases, so s (a + e) and the parts of s rounded up bound it.
__host__ __device__ __forceinline__ int loss_drift(const SeedCosts& c, const Core& k, int loss) {
  const int a = c.a, e = c.ext, cd = c.move2_del, ci = c.move2_ins;
  auto rest = [](int parts, int per) { return parts > 0 ? parts * per : 0; };
  const int l2 = 2 * (loss - c.open);
  const int parts = k.missed + k.hmin;
  int w = paid_bases(l2 - rest(parts - 1, cd), c.per_del);
  int v = inserted_bases(l2, c.per_ins, parts - 2, ci);
  w = v > w ? v : w;
  if (k.hmin > 0) {
    const int s = k.span, d2 = l2 - 2 * (c.open + s * e);
    v = paid_bases(d2 - rest(k.missed - 2, cd), c.per_del);
    w = v > w ? v : w;
    v = inserted_bases(d2, c.per_both, k.missed - 3, ci);
    w = v > w ? v : w;
    v = paid_bases(d2 - 2 * s * (a + e) - rest(k.missed - 3 - (s + kSeed - 3) / kSeed, ci), c.per_del);
    w = v > w ? v : w;
    v = inserted_bases(l2 - 2 * c.open, c.per_ins, k.missed - 4, ci) - s;
    w = v > w ? v : w;
  }
  return w;
}

// What leaving the one diagonal of all occurrences for read bases [from, to]
// with k mismatches there may save, doubled, before its gaps' own loss: each
// part inside is spoiled, but `free` of them, which the gaps (and, local, a
// clipped end) touch.
__host__ __device__ __forceinline__ int leave_saves2(int lose2, int leave2, int T, int from, int to, int k, int free) {
  const int parts = ((to + 1) / kSeed < T ? (to + 1) / kSeed : T) - (from + kSeed - 1) / kSeed - free;
  return lose2 * k - (parts > 0 ? parts * leave2 : 0);
}

// How many times 16 diagonals hold the core and w diagonals on both sides, and
// the diagonals that ns times 16 leave on each.
__host__ __device__ __forceinline__ int band_strips(int span, int w) { return (span + 1 + 2 * w + 15) >> 4; }
__host__ __device__ __forceinline__ int band_margin(int span, int ns) { return (16 * ns - (span + 1)) >> 1; }

}  // namespace mica
