// The bounds of the seeded bands (paper_1402_4876_amd/csrc/seed_bound.h) held
// against full tables, as host code under UndefinedBehaviorSanitizer
// (tests/test_seed_bound.py).
//
// For random legal scorings and read / window pairs built to sit at the
// bounds' edges (window stretches that repeat parts of the read on other
// diagonals, parts without occurrence, long gaps near an end), a full affine-gap
// table gives the best score and, over all alignments that reach it, the lowest
// and the highest diagonal any of them visits.  What the scan would find
// (occurrences of the 12-base parts, the core, the parts without one) is worked
// out here by plain loops.  Checked for each pair:
// - an alignment whose loss is certain to match a part visits the core;
// - the best alignments stay within loss_drift diagonals of the core;
// - where leaving the one diagonal of all occurrences never pays, the best
//   alignment is that diagonal alone;
// - loss_drift grows with the loss.
// Arguments: "local" or "semiglobal", seed, number of pairs.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#define __host__
#define __device__
#define __forceinline__ inline
#include "seed_bound.h"

using namespace mica;

static const int kNone = -(1 << 28);
static const char kLetters[] = "ACGT";

struct Scoring {
  int a, b, o, e;
};

// A score and the diagonals (j - i) of all alignments that reach it.
struct Best {
  int v = kNone, lo = 1 << 20, hi = -(1 << 20);
  void take(const Best& x, int add) {
    if (x.v <= kNone / 2) return;
    const int s = x.v + add;
    if (s > v) {
      v = s;
      lo = x.lo;
      hi = x.hi;
    } else if (s == v) {
      lo = std::min(lo, x.lo);
      hi = std::max(hi, x.hi);
    }
  }
  void visit(int d) {
    if (v <= kNone / 2) return;
    lo = std::min(lo, d);
    hi = std::max(hi, d);
  }
};

// The best alignment of q in w: semi-global (all of q, free window ends) or
// local.  ends: how many cells hold it.
static Best align(const std::vector<int>& q, const std::vector<int>& w, const Scoring& s, bool local, int* ends) {
  const int m = (int)q.size(), n = (int)w.size();
  std::vector<Best> H((size_t)n + 1), I((size_t)n + 1);
  for (int j = 0; j <= n; ++j) {
    H[(size_t)j].v = 0;
    H[(size_t)j].lo = H[(size_t)j].hi = j;
  }
  Best out;
  *ends = 0;
  auto end = [&](const Best& h) {
    if (h.v > out.v) *ends = 0;
    if (h.v == out.v || h.v > out.v) ++*ends;
    out.take(h, 0);
  };
  for (int i = 1; i <= m; ++i) {
    Best diag = H[0], D, zero;
    zero.v = 0;
    Best column;  // all inserted so far
    column.take(H[0], -s.o - s.e);
    column.take(I[0], -s.e);
    column.visit(-i);
    H[0] = I[0] = column;
    if (local) {
      zero.lo = zero.hi = -i;
      H[0].take(zero, 0);
    }
    Best left = H[0];
    for (int j = 1; j <= n; ++j) {
      const int d = j - i;
      Best ins, del, h;
      ins.take(H[(size_t)j], -s.o - s.e);
      ins.take(I[(size_t)j], -s.e);
      ins.visit(d);
      del.take(left, -s.o - s.e);
      del.take(D, -s.e);
      del.visit(d);
      h.take(diag, q[(size_t)i - 1] == w[(size_t)j - 1] ? s.a : s.b);
      h.take(ins, 0);
      h.take(del, 0);
      h.visit(d);
      if (local) {
        zero.lo = zero.hi = d;
        h.take(zero, 0);
      }
      diag = H[(size_t)j];
      H[(size_t)j] = h;
      I[(size_t)j] = ins;
      D = del;
      left = h;
      if (local && h.v > 0) end(h);
    }
    if (i == m && !local)
      for (int j = 0; j <= n; ++j) end(H[(size_t)j]);
  }
  return out;
}

// What the scan finds.
struct Found {
  bool usable = false;  // no two equal parts, an occurrence, a core within 64 diagonals
  int T = 0, c0 = 0, c1 = 0;
  Core core{0, 0, 0};
};
static Found scan(const std::vector<int>& q, const std::vector<int>& w, bool local) {
  const int m = (int)q.size(), n = (int)w.size();
  Found f;
  f.T = m / kSeed;
  auto same = [](const int* x, const int* y) { return std::equal(x, x + kSeed, y); };
  for (int s = 0; s < f.T; ++s)
    for (int t = s + 1; t < f.T; ++t)
      if (same(&q[(size_t)(kSeed * s)], &q[(size_t)(kSeed * t)])) return f;
  std::vector<std::pair<int, int>> hits;  // diagonal, part
  std::vector<bool> has((size_t)std::max(f.T, 1));
  for (int p = 0; p + kSeed <= n; ++p)
    for (int s = 0; s < f.T; ++s)
      if (same(&w[(size_t)p], &q[(size_t)(kSeed * s)])) {
        hits.push_back({p - kSeed * s, s});
        has[(size_t)s] = true;
      }
  if (hits.empty()) return f;
  f.c0 = std::min_element(hits.begin(), hits.end())->first;
  f.c1 = std::max_element(hits.begin(), hits.end())->first;
  f.core.span = f.c1 - f.c0;
  if (f.core.span >= 64) return f;
  f.usable = true;
  int occur = 0;
  for (int s = 0; s < f.T; ++s) {
    occur += has[(size_t)s] ? 1 : 0;
    if (!has[(size_t)s] && !(local && (s == 0 || s == f.T - 1))) f.core.missed++;
  }
  if (f.core.span > 0 && (int)hits.size() == occur) {
    int on0 = 0, on1 = 0, at0 = 0, at1 = 0;
    for (const auto& h : hits) {
      const int counts = local && (h.second == 0 || h.second == f.T - 1) ? 0 : 1;
      on0 += h.first == f.c0 ? 1 : 0;
      on1 += h.first == f.c1 ? 1 : 0;
      at0 += h.first == f.c0 ? counts : 0;
      at1 += h.first == f.c1 ? counts : 0;
    }
    if (on0 + on1 == (int)hits.size()) f.core.hmin = std::min(at0, at1);
  }
  return f;
}

// Is the one diagonal of all occurrences certain to be the only best alignment?
static bool stays(const std::vector<int>& q, const std::vector<int>& w, const Scoring& s, const SeedCosts& c, bool local,
                  const Found& f, int* score) {
  const int m = (int)q.size(), n = (int)w.size();
  if (f.core.span > 0 || f.c0 < 0 || f.c0 + m > n) return false;
  std::vector<int> hit;
  for (int i = 0; i < m; ++i)
    if (q[(size_t)i] != w[(size_t)(i + f.c0)]) hit.push_back(i);
  const int k = (int)hit.size(), gap2 = 2 * (s.o + s.e), lose2 = 2 * (s.a - s.b);
  const int leave2 = local ? c.leave2_local : c.leave2;
  for (int i = 0; i < k; ++i) {
    const int p = hit[(size_t)i];
    int head = leave_saves2(lose2, leave2, f.T, 0, p, i + 1, local ? 2 : 1);
    int tail = leave_saves2(lose2, leave2, f.T, p, m - 1, k - i, local ? 2 : 1);
    if (local) {
      head = std::min(head, 2 * s.a * (p + 1));
      tail = std::min(tail, 2 * s.a * (m - p));
    }
    if (head >= gap2 || tail >= gap2) return false;
    for (int j = i; j < k; ++j)
      if (leave_saves2(lose2, leave2, f.T, p, hit[(size_t)j], j - i + 1, 2) >= 2 * gap2) return false;
  }
  if (local) {
    int h = 0, best = 0;
    for (int i = 0; i < m; ++i) {
      h = std::max(0, h + (q[(size_t)i] == w[(size_t)(i + f.c0)] ? s.a : s.b));
      best = std::max(best, h);
    }
    *score = best;
  } else {
    *score = s.a * m - (s.a - s.b) * k;
  }
  return loss_certain(c, local, f.T, s.a * m - *score);
}

static int failures = 0, certified = 0, edge = 0, direct = 0, cored = 0;

static std::string letters(const std::vector<int>& v) {
  std::string s;
  for (int x : v) s += kLetters[x];
  return s;
}

static void report(const char* what, const std::vector<int>& q, const std::vector<int>& w, const Scoring& s,
                   const Found& f, const Best& b, int drift) {
  if (++failures > 5) return;
  std::printf("%s: scoring (%d,%d,%d,%d) score %d diagonals %d..%d core %d..%d hmin %d missed %d drift %d\n  %s\n  %s\n", what,
              s.a, s.b, s.o, s.e, b.v, b.lo, b.hi, f.c0, f.c1, f.core.hmin, f.core.missed, drift, letters(q).c_str(),
              letters(w).c_str());
}

static void check(const std::vector<int>& q, const std::vector<int>& w, const Scoring& s, bool local) {
  const int m = (int)q.size();
  const Found f = scan(q, w, local);
  if (!f.usable) return;
  ++cored;
  const SeedCosts c = seed_costs(s.a, s.b, s.o, s.e, 85);
  int ends = 0;
  const Best b = align(q, w, s, local, &ends);
  if (b.v <= 0 && local) return;
  const int loss = s.a * m - b.v;
  if (!loss_certain(c, local, f.T, loss)) return;
  ++certified;
  const int drift = loss_drift(c, f.core, loss);
  if (b.lo > f.c1 || b.hi < f.c0) report("no part matched", q, w, s, f, b, drift);
  if (b.lo < f.c0 - drift || b.hi > f.c1 + drift) report("outside the band", q, w, s, f, b, drift);
  edge += drift > 0 && (b.lo == f.c0 - drift || b.hi == f.c1 + drift) ? 1 : 0;
  for (int up = 1; up < 40; up += 13)
    if (loss_drift(c, f.core, loss + up) < drift) report("not monotone", q, w, s, f, b, drift);
  int score = 0;
  if (stays(q, w, s, c, local, f, &score)) {
    ++direct;
    if (score != b.v || b.lo != f.c0 || b.hi != f.c0) report("leaves its diagonal", q, w, s, f, b, drift);
  }
}

// Pairs whose best alignment a weaker bound missed: long insertions that
// swallow parts; end parts, which clipping spoils, on a diagonal of their own.
struct Known {
  bool local;
  Scoring s;
  const char *read, *window;
};
static const Known known[] = {
    {false, {2, -20, 40, 2},
     "TCAGTTTATGCCCCCGTAGGCCCTAGTAGTATGCCAAGGCGTGCTTTCCTCCTCCCTTACTATGCAAACGCTCTGCAGATTTCGTCCAGATGCATATTGCGTCCG",
     "GTATGAAACGTTGTTCAGTTTATGCCCCCGTAGGCCCTAGTAGTATGCCAAGGCGTGCTTTCCTCCTCCCTTACTATGCAAACGCGATGCATATTGCGTCCGGATGCATATTGC"
     "GTCCGGAAGACTCGAGTT"},
    {false, {1, -9, 16, 2},
     "CCGTCCGGGACTCGCTTCGAAGATTAGTCGCGTGGCCTCTGGTAAATAGATTAATGTAACCATGTCCGTAACTTTTTACCGTAACCCTTTTCTACCGTAACCCTT",
     "CGACCTCGGATCACATTGGAAGGTCCCGTCCGGGACTCGCTTCGAAGATTAGTCGCGTGGCCTCTGGTAAATAGATTAATGTAACCATGTCCGTAATTTTCTACCGTAACCCTT"
     "TCCTACCGTGTCCAATCATCTGTCAGTGACGCTAGAGTATTAT"},
    {false, {1, -23, 18, 2},
     "CTCGTCTAAATCATCTTCTCGTCTAAACGATATTTCTCCGGCTGAGTGGTCATAAGGCAGCTTTTGTTCGGAGTGTATGCCACCTCATACCGATAGTCTAGGGTGGGATAGATG"
     "CTTCGATGCTATAGCGAGCGTAACGGAGC",
     "CCGATGTATTCTAATACACCGCGAGTATCTCGACTAAATCATCTGCTCGTCTAAATGATATTTCTCCGGCTGAGTGGTCATAAGGCAGCTTTTGTTCGGAGTGTATGCCACCTC"
     "ATACCGATAGTCTAGGGTGGGATAGATGCTTCGATGCTATAGCGAGCGTAACGGAGCGAGAGCTTGGAC"},
    {true, {1, -4, 6, 1},
     "ATGTTGCGCCCGTGTAATCCTGGCTAAAAATATAGGACACACACCGCCAGGTCGGTGAACTCATCGCGACTGCGGATCTACCCTTTATCGTACCGTCTCTTATTTTGATATCGT"
     "ACCGTCCTG",
     "TAGACTTTCTATGCCTTCACAGGCCCTGGACCATGAGAAAGATAGCCATGTTGCGCCCGCTAATTGGAGGTTGTTGCGCCCGTGTAATCCTGGCTAAAAATATAGGACACACAC"
     "CGCCAGGTCGGTGAACTCATCGCGACTGCGGATCTACCCTTTATCGTACCGTCTCTTATTTTGATAGGATAATCGTACCGTCCTGAAACTAAGTGCGAACAG"},
};

int main(int argc, char** argv) {
  if (argc < 4) return 2;
  const bool local = std::strcmp(argv[1], "local") == 0;
  std::mt19937_64 rng((uint64_t)std::atoll(argv[2]));
  const long pairs = std::atol(argv[3]);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (uint64_t)(hi - lo + 1)); };
  for (const Known& k : known) {
    std::vector<int> q, w;
    for (const char* x = k.read; *x; ++x) q.push_back((int)(std::strchr(kLetters, *x) - kLetters));
    for (const char* x = k.window; *x; ++x) w.push_back((int)(std::strchr(kLetters, *x) - kLetters));
    if (k.local == local) check(q, w, k.s, local);
  }
  static const Scoring common[] = {{1, -4, 6, 1}, {2, -4, 4, 2}, {1, -3, 5, 2}, {1, -1, 20, 1}, {1, -9, 16, 2}};
  for (long r = 0; r < pairs; ++r) {
    Scoring s = common[rng() % 5];
    if (pick(0, 2)) s = Scoring{pick(1, pick(0, 3) ? 2 : 6), -pick(0, pick(0, 1) ? 6 : 30), pick(0, pick(0, 1) ? 8 : 60), pick(1, pick(0, 2) ? 2 : 6)};
    const int m = pick(pick(0, 1) ? 36 : 80, 160), flank = pick(0, 40);
    std::vector<int> q((size_t)m);
    for (int& x : q) x = pick(0, 3);
    if (pick(0, 3) == 0) {  // a stretch of the read repeats, not quite
      const int len = pick(12, std::min(40, m / 2)), from = pick(0, m - len), to = pick(0, m - len);
      for (int i = 0; i < len; ++i)
        if (pick(0, 9)) q[(size_t)(to + i)] = q[(size_t)(from + i)];
    }
    std::vector<int> w((size_t)(m + 2 * flank + pick(0, 20)));
    for (int& x : w) x = pick(0, 3);
    // stretches of the read laid over the window: the whole read at the flank,
    // then others beside it, each with mutations of their own
    auto lay = [&](int from, int to, int d, int one_in) {
      for (int i = from; i < to; ++i) {
        const int j = i + d;
        if (j < 0 || j >= (int)w.size()) continue;
        w[(size_t)j] = one_in && pick(1, one_in) == 1 ? (q[(size_t)i] + pick(1, 3)) & 3 : q[(size_t)i];
      }
    };
    static const int rates[] = {0, 8, 12, 16, 25, 60};
    lay(0, m, flank, pick(0, 2) ? 0 : rates[rng() % 6]);
    for (int t = pick(0, 3); t > 0; --t) {
      const int len = pick(3, pick(0, 1) ? 25 : m);
      const int from = pick(0, 2) ? (pick(0, 1) ? 0 : std::max(0, m - len)) : pick(0, m - 1);
      int d = pick(0, 1) ? pick(-5, 5) : pick(-40, 40);
      if (pick(0, 3) == 0) d = 0;
      lay(from, std::min(m, from + len), flank + d, pick(0, 1) ? 0 : rates[rng() % 6]);
    }
    // parts without occurrence: a substitution in each of some neighbours
    if (pick(0, 1)) {
      const int T = m / kSeed, first = pick(0, T - 1), count = pick(1, 6);
      for (int k = first; k < T && k < first + count; ++k) {
        const int j = kSeed * k + pick(0, kSeed - 1) + flank;
        if (j < (int)w.size()) w[(size_t)j] = (w[(size_t)j] + pick(1, 3)) & 3;
      }
    }
    // an end of the read beside its place, with parts without occurrence next
    // to it: what a long gap near that end would win
    if (pick(0, 2) == 0) {
      const int len = pick(6, 45), d = pick(0, 1) ? pick(8, 40) : -pick(8, 40);
      const bool tail = pick(0, 1);
      const int from = tail ? std::max(0, m - len) : 0, to = tail ? m : std::min(m, len);
      lay(from, to, flank + d, 0);
      const int spoil = kSeed * pick(1, 5);
      for (int i = tail ? std::max(0, from - spoil) : 0; i < (tail ? m : std::min(m, to + spoil)); i += pick(kSeed / 2, kSeed)) {
        const int j = i + flank;
        const bool copy = j >= from + flank + d && j < to + flank + d;
        if (j < (int)w.size() && !copy) w[(size_t)j] = (w[(size_t)j] + pick(1, 3)) & 3;
      }
    }
    if (pick(0, 2) == 0) {  // a gap
      const int at = pick(0, (int)w.size() - 1), len = pick(1, 25);
      if (pick(0, 1)) w.erase(w.begin() + at, w.begin() + std::min((int)w.size(), at + len));
      else for (int i = 0; i < len; ++i) w.insert(w.begin() + at, pick(0, 3));
    }
    if ((int)w.size() >= kSeed) check(q, w, s, local);

    // the read in its place but for the first and the last part, which lie on a
    // diagonal of their own (one of them as the read repeats it further in), and
    // an end without its part beside
    if (r % 4) continue;
    const int T = m / kSeed, last = kSeed * (T - 1);
    const int d = pick(0, 1) ? pick(1, 30) : -pick(1, 30);
    for (int i = 0; i < kSeed; ++i) {
      const int from = d > 0 ? i : last + i;
      if (from + d >= 0 && from + d < m) q[(size_t)(from + d)] = q[(size_t)from];
    }
    s = common[rng() % 5];
    w.assign((size_t)(m + 120), 0);
    for (int& x : w) x = pick(0, 3);
    lay(0, m, 60, 0);
    for (int part : {0, last})
      for (int t = pick(1, 3); t > 0; --t) {
        int& x = w[(size_t)(60 + part + pick(0, kSeed - 1))];
        x = (x + pick(1, 3)) & 3;
      }
    if (d > 0) lay(last, last + kSeed, 60 + d, 0);
    else lay(0, kSeed, 60 + d, 0);
    const int past = pick(0, 1) ? pick(1, 12) : -pick(1, 12);
    if (pick(0, 1)) lay(last + pick(1, 4), m, 60 + past, 0);
    else lay(0, kSeed - pick(1, 4), 60 + past, 0);
    check(q, w, s, local);
  }
  std::printf("%ld pairs: %d with a core, %d certain, %d at the edge, %d without a gap, %d failures\n", pairs, cored, certified,
              edge, direct, failures);
  return failures ? 1 : 0;
}
