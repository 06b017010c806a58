// Seeded band alignment (included by dp_fill.h's users after it): pairs whose
// whole answer provably lies in a narrow band of diagonals are finished here,
// before the fills, without computing the rest of their tables.
//
// What is proven.  Call a m - score the loss of an alignment of a read of m
// bases, a the match score, and cut the read into T = m / kSeed parts of kSeed
// bases.  An alignment in which no part is matched exactly along one diagonal
// spoils every part, and spoiling k parts costs at least k c (seed_bound.h; in
// local mode the two clipped ends may spoil one part each for free).  So an
// alignment of loss L < T c runs through an exact occurrence of some part.
// The scan finds all occurrences of all parts in the window, every position
// against every part; the diagonals c0..c1 they span are the pair's core.
//
// Bands.  A part without any occurrence is spoiled in every alignment, so an
// alignment that also moves w diagonals off the core loses the deleted or
// inserted bases of that move, its gap open, and c for every such part that
// the move's own runs do not spoil.  With occurrences on exactly two diagonals
// s apart, h of them at least on each, an alignment through both pays that gap
// too, and one through a single diagonal spoils the other's h parts as well.
// X(L) is the largest w this leaves for a loss L (loss_drift, with the cases).
// If a band holds X(L) diagonals on both sides of the core, where L < T c is
// the loss of the best alignment inside it, then every alignment that scores
// as much lies in the band: score, end cell and its ties are the full
// table's, and so is the traceback (the argument of band.h).  An extension
// starts on diagonal 0 by definition and needs no parts: the best prefix of
// that diagonal bounds its loss, and the band follows.
//
// No gap.  With all occurrences on one diagonal of k mismatches, an
// alignment that leaves it for good (or joins it late) pays a gap and, off
// it, one spoiled part's cost c for every part but the one the gap touches,
// and saves the mismatches of that stretch; one that leaves it and returns
// pays two gaps.  When that is a loss for every stretch of mismatches, the
// diagonal is the only best alignment and is written out at once.
//
// A pair without an occurrence (unrelated read and window), with too wide a
// band, with a loss the parts cannot certify or with two equal parts is left
// to the fills, unchanged.
//
// Four kernels.  k_seed_sample: in large batches for which looking may not pay,
// whether it does.  k_seed_scan: a wave scans 8 pairs, answers those without a
// gap, and lists the others with their band; it needs few registers, so many
// waves hide its chain of dependent loads.  k_seed_band: the listed bands, 8
// pairs (4 in 32 bits) to a wave, the wide ones first; a band that turns out
// too narrow is aligned again in a wider one by the same wave.  k_seed_left:
// the full traceback of the pairs left, where there are few.
//
// What bounds them: VALU instructions (scan 390, bands 603 per pair of 10^6
// reads of 150 in windows of 400, of which 57% are answered by the scan and
// 0.1% left; the full table takes 6,460) and, in small batches, the latency
// of one band (60 us for 48 pairs of 76 to 151 bases).  10^6 x 150 x 400: scan
// 0.70 ms, bands 1.35 ms, left pairs 0.12 ms, in place of 10.7 ms of fills and
// 1.3 ms of side lists.
#pragma once

#include "dp_fill.h"
#include "plan_scan.h"

namespace mica {

// Resident waves per SIMD.
constexpr int kScanWaves = 6;
// pairs that keep the GPU busy for more than an item's time
constexpr int kBusyPairs = 16384;
constexpr int kDearWindow = 768;
constexpr int kBandWaves = 4;

// The scan's LDS words of a pair before its window and read: {lowest, highest
// diagonal, occurrences, -, parts that occur (3 words), -}, the diagonals of
// the first 16 occurrences.
constexpr int kPrHits = 16;
constexpr int kPrPair = 8 + kPrHits;
// And of a wave: the pairs it will add to the four lists (left, bands of up to
// 16, 32 and 64 diagonals).
constexpr int kPrOutOff = 8 * kPrPair;
constexpr int kPrOut = kPruneItem * kScanChunk;
static_assert(kPrOutOff + 4 * kPrOut == kScanStaticWords, "the host sizes the LDS by this");
// A band kernel's: the item's pairs and the pairs to align again, an entry
// {pair, band, core} each.
constexpr int kBandItem = 8;
constexpr int kBandAgain = 16;  // of up to 32 diagonals, and as many of up to 64
constexpr int kBandEntry = 3;
static_assert((kBandItem + 2 * kBandAgain) * kBandEntry <= kBandStaticWords, "the host sizes the LDS by this");

// A listed pair's band: lowest diagonal, diagonals on both sides of the core
// (kProven: nothing to check afterwards), width in 16 diagonals.
constexpr int kProven = 255;
__device__ __forceinline__ uint32_t band_word(int lo, int margin, int ns) {
  return ((uint32_t)(lo + 32768) & 0xFFFFu) | ((uint32_t)margin << 16) | ((uint32_t)ns << 24);
}

// word w of 16 bases of a stretch that starts at base `at`, from 2-bit words
// (reads no word past `last`, the array's last one)
__device__ __forceinline__ uint32_t stretch_word(const MICA_GLOBAL uint32_t* __restrict__ seq, uint64_t at, int w,
                                                 uint64_t last) {
  const uint64_t p = at + (uint64_t)w * 16u;
  const uint64_t i = p >> 4;
  const uint32_t lo = seq[i < last ? i : last];
  const uint32_t hi = seq[i + 1 < last ? i + 1 : last];
  return __builtin_amdgcn_alignbit(hi, lo, 2u * (uint32_t)(p & 15u));
}
// 16 bases from a position on that may lie before the array's first base or
// past its last one (those bases are arbitrary)
__device__ __forceinline__ uint32_t signed_word(const MICA_GLOBAL uint32_t* __restrict__ seq, int64_t at,
                                                uint64_t last) {
  const int64_t i = at >> 4;
  const uint64_t a = i < 0 ? 0 : ((uint64_t)i < last ? (uint64_t)i : last);
  const uint64_t b = i + 1 < 0 ? 0 : ((uint64_t)(i + 1) < last ? (uint64_t)(i + 1) : last);
  return __builtin_amdgcn_alignbit(seq[b], seq[a], 2u * (uint32_t)(at & 15));
}
// the same from a stretch's words in LDS, at any base
__device__ __forceinline__ uint32_t lds_bases(const uint32_t* words, int p) {
  return __builtin_amdgcn_alignbit(words[(p >> 4) + 1], words[p >> 4], 2u * (uint32_t)(p & 15));
}

// max / min / sum over the 8 lanes of a pair
__device__ __forceinline__ int max8(int v) {
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) {
    const int o = __shfl_xor(v, d, 64);
    v = o > v ? o : v;
  }
  return v;
}
__device__ __forceinline__ int min8(int v) { return -max8(-v); }
__device__ __forceinline__ int sum8(int v) {
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// The values every band item of a pair needs to be able to hold in 16 bits:
// the largest score plus the deletion scan's lane offsets, the least less the
// dummy rows of the band fill.
template <class V>
__device__ __forceinline__ bool band_fits(const Params* __restrict__ prm, int m, int n, int h0) {
  if constexpr (V::kPairs == 1) return true;
  const long top = (long)h0 + (long)prm->sa * (m < n ? m : n);
  const long off = 64L * prm->se + prm->so;
  // (the least value of a cell, and kMaxM dummy rows)
  const long low = 2L * prm->so + (long)(m + 1) * prm->se + kMaxM;
  return top + off <= 32767 && off <= 32767 && low <= 32767;
}

// The list of the pairs left and the list of bands, each in a bucket's range:
// the two lists the fills use later, the left pairs in the one they are read
// from (left_full of the planner).  Bands of up to 16 diagonals go from the
// start of the range up, of up to 32 from its end down, wider ones to a list of
// their own; their bands and cores lie in arrays by pair that are free between
// the planner and the fills.
template <int MODE, bool TRACE>
__device__ __forceinline__ MICA_GLOBAL uint32_t* left_list(const Params* __restrict__ prm) {
  return G(TRACE && left_full(prm, MODE) ? prm->fbsorted : prm->sorted);
}
template <int MODE, bool TRACE>
__device__ __forceinline__ MICA_GLOBAL uint32_t* band_list(const Params* __restrict__ prm) {
  return G(TRACE && left_full(prm, MODE) ? prm->sorted : prm->fbsorted);
}
// Adds the pairs of the lanes with `mine` to list li (0 left, then the bands by
// width) of the wave's output.
__device__ __forceinline__ void put_out(uint32_t* lds, int li, int* cnt, bool mine, uint32_t p) {
  const uint64_t bal = __ballot(mine);
  if (mine) {
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
    lds[kPrOutOff + li * kPrOut + *cnt + (int)rank] = p;
  }
  *cnt += __builtin_popcountll(bal);
}
// The count of a bucket's list li.
__device__ __forceinline__ uint32_t* out_count(const Params* __restrict__ prm, int li, int bucket) {
  return (li == 0 ? prm->rcount : (li == 1 ? prm->nbcount : (li == 2 ? prm->w32count : prm->w64count))) + bucket;
}
// Moves the wave's output to the bucket's lists, from entry b[li] of list li.
template <int MODE, bool TRACE>
__device__ __forceinline__ void write_out(const Params* __restrict__ prm, int bucket, const uint32_t* lds,
                                          const int cnt[4], const uint32_t b[4]) {
  const int lane = threadIdx.x & 63;
  const uint32_t bs = G(prm->bstart)[bucket];
  const uint32_t* out = lds + kPrOutOff;
  if (lane < cnt[0]) left_list<MODE, TRACE>(prm)[bs + b[0] + lane] = out[lane];
  if (lane < cnt[1]) band_list<MODE, TRACE>(prm)[bs + b[1] + lane] = out[kPrOut + lane];
  if (lane < cnt[2]) band_list<MODE, TRACE>(prm)[bs + G(prm->bcount)[bucket] - 1u - b[2] - lane] = out[2 * kPrOut + lane];
  if (lane < cnt[3]) G(prm->wlist)[bs + b[3] + lane] = out[3 * kPrOut + lane];
}
template <bool TRACE>
__device__ __forceinline__ void write_out(const Params* __restrict__ prm, int mode, int bucket, const uint32_t* lds,
                                          const int cnt[4], const uint32_t b[4]) {
  if (mode == 0) write_out<0, TRACE>(prm, bucket, lds, cnt, b);
  else if (mode == 1) write_out<1, TRACE>(prm, bucket, lds, cnt, b);
  else write_out<2, TRACE>(prm, bucket, lds, cnt, b);
}
// The scan of an item of up to 8 pairs of one mode, pair p of 8 lanes where
// they are valid.  SAMPLE: only how many of them it would answer or list for a
// band, and the table cells this saves less its own cost (saved).  10^6 pairs of
// 150 x 400 take 10.7 ms in the fill, 0.18 us per 1,000 cells; a pair's scan as
// long as 1,400 cells and 5% of the table, a row of a band of 16 diagonals as
// long as 112 columns (scores alone 90), of 32 and 64 two and four times that.
// A traced pair refills its band, some 64 columns, and may pass through a side
// list, a tenth of the time more (local, whose cells are dearer too, half).
template <class V, int MODE, bool TRACE, bool SAMPLE>
__device__ __forceinline__ int prune_scan(const Params* __restrict__ prm, bool valid, int p, uint32_t* lds, int* cnt,
                                          BandCount* count, int* saved = nullptr) {
  constexpr bool EXT = (MODE == 2);
  constexpr bool LOCAL = (MODE == 1);
  const int lane = threadIdx.x & 63;
  const int q = lane >> 3, x = lane & 7;
  const int sa = prm->sa, sb = prm->sb, so = prm->so, se = prm->se;
  const MICA_GLOBAL uint32_t* __restrict__ ref2b = G(prm->ref2b);
  const MICA_GLOBAL uint32_t* __restrict__ reads2b = G(prm->reads2b);
  const int WN = prm->pr_win_words, RN = prm->pr_read_words, TN = prm->pr_part_words;
  uint32_t* const win = lds + kScanStaticWords;
  uint32_t* const rd = win + 8 * WN;
  uint32_t* const part = rd + 8 * RN;
  int* const res = (int*)lds + q * kPrPair;
  int* const hit = res + 8;

  int m = 0, n = 0, h0 = 0;
  uint64_t wo = 0, ro = 0;
  if (valid) {
    m = G(prm->read_len)[p];
    n = G(prm->win_len)[p];
    wo = G(prm->win_off)[p];
    ro = G(prm->read_off)[p];
    if constexpr (EXT) h0 = prm->ext_h0 ? G(prm->ext_h0)[p] : prm->ext_default_h0;
  }
  const int T = EXT ? 0 : m / kSeed;
  // an extension looks at the window's part beside diagonal 0 only
  const int nl = EXT ? (n < m ? n : m) : n;
  const int nw = (nl + 15) >> 4, mw = (m + 15) >> 4;
  const uint64_t ref_last = (prm->ref_len - 1) >> 4, reads_last = (prm->reads_len - 1) >> 4;
  if (valid) {
    for (int w = x; w < nw + 2; w += 8) win[q * WN + w] = w < nw ? stretch_word(ref2b, wo, w, ref_last) : 0u;
    for (int w = x; w < mw + 1; w += 8) rd[q * RN + w] = w < mw ? stretch_word(reads2b, ro, w, reads_last) : 0u;
  }
  if (x == 0) {
    res[0] = 0x7FFFFFFF;
    res[1] = -0x7FFFFFFF;
    res[2] = 0;
    res[4] = res[5] = res[6] = 0;
  }
  lds_wait();

  bool twin = false;  // two equal parts: an occurrence would not name its part
  if constexpr (!EXT) {
    const int tmax = (wave_max_int(T) + 3) & ~3;
    // part s in the high 24 bits, its number below.  Pads up to tmax have
    // numbers past T, which the reader ignores, and a number below 256 with
    // equal bases never loses to one.
    uint32_t* const pq = part + q * TN;
    for (int s = x; s < tmax; s += 8) pq[s] = s < T ? (lds_bases(rd + q * RN, kSeed * s) << 8) | (uint32_t)s : 0xFFFFFF00u | (uint32_t)s;
    lds_wait();
    // each part against every other (pads of equal bases count too: such a
    // pair is only left to the fills)
    for (int s = x; s < tmax; s += 8) {
      const uint32_t k = pq[s];
      int same = 0;
      for (int s2 = 0; s2 < tmax; s2 += 4)
#pragma unroll
        for (int u = 0; u < 4; ++u) same += (k ^ pq[s2 + u]) < 256u ? 1 : 0;
      twin |= s < T && same > 1;
    }
    twin = (__ballot(twin) >> (8 * q) & 0xFFu) != 0;
    // positions p0 .. p0 + kSeed - 1 of the pair's window, a "tile" per lane;
    // first for four parts: where none of the item's pairs has one of them,
    // the others are not looked for
    // (reads of tandem repeats would have occurrences everywhere)
    const int tiles = valid && T > 0 && !twin ? n / kSeed : 0;  // of the n - kSeed + 1 positions
    const int rounds = (wave_max_int(tiles) + 7) >> 3;
    bool any = false;
    for (int from = 0, to = 4; from < tmax; from = to, to = tmax) {
      for (int r = 0; r < rounds; ++r) {
        const int tile = x + 8 * r;
        const bool live = tile < tiles;
        const int p0 = live ? kSeed * tile : 0;
        const uint32_t* wq = win + q * WN + (p0 >> 4);
        const uint32_t sh = 2u * (uint32_t)(p0 & 15);
        const uint32_t w1 = wq[1];
        const uint32_t lo = __builtin_amdgcn_alignbit(w1, wq[0], sh);
        const uint32_t hi = __builtin_amdgcn_alignbit(wq[2], w1, sh);
        // positions past the last one that holds a whole part never match
        const int left = live ? n - kSeed + 1 - p0 : 0;
        uint32_t km[kSeed], z[kSeed];
        static_for<kSeed>([&](auto tc) {
          constexpr int t = decltype(tc)::value;
          km[t] = __builtin_amdgcn_alignbit(hi, lo, 2 * t) << 8;
          z[t] = 0xFFFFFFFFu;
        });
        for (int s = from; s < to; s += 4) {
          const uint32_t s0 = pq[s], s1 = pq[s + 1], s2 = pq[s + 2], s3 = pq[s + 3];
          static_for<kSeed>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            const uint32_t x0 = km[t] ^ s0, x1 = km[t] ^ s1, x2 = km[t] ^ s2, x3 = km[t] ^ s3;
            uint32_t v = x0 < x1 ? x0 : x1;
            v = v < z[t] ? v : z[t];
            uint32_t u = x2 < x3 ? x2 : x3;
            z[t] = u < v ? u : v;
          });
        }
        static_for<kSeed>([&](auto tc) {
          constexpr int t = decltype(tc)::value;
          if (z[t] < (uint32_t)T && t < left) {
            const int d = p0 + t - kSeed * (int)z[t];
            any = true;
            atomicMin(&res[0], d);
            atomicMax(&res[1], d);
            const int at = atomicAdd(&res[2], 1);
            // (local: whether it is the first or the last part in the low bit)
            if (at < kPrHits) hit[at] = LOCAL ? 2 * d + (z[t] == 0 || (int)z[t] == T - 1 ? 1 : 0) : d;
            atomicOr((uint32_t*)&res[4 + (z[t] >> 5)], 1u << (z[t] & 31u));
          }
        });
      }
      if (__ballot(any) == 0) {  // none of these pairs
        if constexpr (SAMPLE) *saved = 0;
        else put_out(lds, 0, &cnt[0], valid && x == 0, (uint32_t)p);
        lds_wait();
        return 0;
      }
    }
    lds_wait();
  }

  // ---- what the scan says of each pair (the same in its 8 lanes) -------------
  bool ok = valid && !twin && band_fits<V>(prm, m, n, h0) && (EXT || T > 0);
  int c0 = 0, hits = 0, missed = 0;
  Core core{0, 0, 0};
  if constexpr (!EXT) {
    c0 = res[0];
    const int c1 = res[1];
    hits = res[2];
    ok = ok && hits > 0 && c1 - c0 < 64;
    core.span = ok ? c1 - c0 : 0;
    const uint32_t m0 = (uint32_t)res[4], m1 = (uint32_t)res[5], m2 = (uint32_t)res[6];
    missed = T - (__builtin_popcount(m0) + __builtin_popcount(m1) + __builtin_popcount(m2));
    core.missed = missed;
    if constexpr (LOCAL) {
      const uint32_t last = (T - 1) < 32 ? m0 >> (T - 1) : (T - 1 < 64 ? m1 >> (T - 33) : m2 >> (T - 65));
      core.missed -= (m0 & 1u) ? 0 : 1;
      core.missed -= (last & 1u) ? 0 : 1;
    }
    // (a part that occurs on both diagonals is spoiled by neither, and in local
    // mode the first and the last are spoiled by clipping)
    if (ok && core.span > 0 && hits <= kPrHits && hits == T - missed) {
      int at0 = 0, at1 = 0;  // occurrences, and of the parts that count from bit 8
#pragma unroll
      for (int u = 0; u < kPrHits / 8; ++u) {
        const int k = x + 8 * u;
        const int v = k < hits ? hit[k] : (LOCAL ? 2 : 1) * (c0 + 1000);
        const int d = LOCAL ? v >> 1 : v;
        const int one = LOCAL && (v & 1) ? 1 : 0x101;
        at0 += d == c0 ? one : 0;
        at1 += d == c1 ? one : 0;
      }
      at0 = sum8(at0);
      at1 = sum8(at1);
      const int h0 = at0 >> 8, h1 = at1 >> 8;
      core.hmin = (at0 & 0xFF) + (at1 & 0xFF) == hits ? (h0 < h1 ? h0 : h1) : 0;
    }
  }
  // mismatches on the one diagonal, where it lies inside the window; their
  // read bases (the first 16) go to the list of occurrences
  const bool one = ok && (EXT ? n >= m : (core.span == 0 && c0 >= 0 && c0 + m <= n));
  const bool look = ok && (EXT || one);
  int mism = 0, best = h0;  // best (extension): the best prefix of diagonal 0
  int total = 0, dense = 0;  // all mismatches, and those of words full of them
  lds_wait();
  {
    const int len = EXT ? nl : m;
    const int rounds = wave_max_int(look ? (len + 127) >> 7 : 0);
    for (int r = 0; r < rounds; ++r) {
      const int w = x + 8 * r;
      uint32_t d = 0;
      int bases = 0;
      if (look && 16 * w < len) {
        const uint32_t v = rd[q * RN + w] ^ lds_bases(win + q * WN, c0 + 16 * w);
        d = (v | (v >> 1)) & 0x55555555u;
        bases = len - 16 * w;
        if (bases < 16) d &= (1u << (2 * bases)) - 1u;
      }
      const int c = __builtin_popcount(d);
      const bool full = !EXT && (c > 4 || 2 * c > bases);
      int incl = full ? c * 0x10001 : c;
#pragma unroll
      for (int s = 1; s < 8; s <<= 1) {
        const int o = __shfl_up(incl, s, 8);
        if (x >= s) incl += o;
      }
      int k = mism + (incl & 0xFFFF) - c;
      if constexpr (EXT) {
        if (look && 16 * w < len) {
          const int v = h0 + sa * (len < 16 * w + 16 ? len : 16 * w + 16) - (sa - sb) * (k + c);
          best = v > best ? v : best;
        }
      }
      // (a word with more than four mismatches is no answer, and its later
      // prefixes are hardly the best)
      if (!EXT && c > 4) k += kPrHits;
      const bool many = (__ballot(!EXT && c > 4) >> (8 * q) & 0xFFu) != 0;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (d == 0) break;
        const int at = 16 * w + (__builtin_ctz(d) >> 1);
        d &= d - 1;
        if constexpr (EXT) {
          const int v = h0 + sa * at - (sa - sb) * k;
          best = v > best ? v : best;
        }
        if (k < kPrHits) hit[k] = at;
        ++k;
      }
      const int sum = __shfl(incl, 7, 8);
      mism += (sum & 0xFFFF) + (many ? kPrHits + 1 : 0);
      if constexpr (!EXT) {
        total += sum & 0xFFFF;
        dense += sum >> 16;
      }
    }
    if constexpr (EXT) best = max8(best);
  }
  lds_wait();

  // ---- no gap possible: the diagonal is the answer ----------------------------
  const int gap = so + se;  // the least loss of a gap
  // whether a band that fails costs more than it might save: not where a table is
  // several bands' worth, nor in a batch of one item's time
  const bool busy = prm->n_pairs >= kBusyPairs && n < kDearWindow;
  const bool known = !EXT && one && mism <= kPrHits;  // every mismatch's place
  bool direct = false;
  int score = 0, ie = 0, i0 = 0, crowd = 0;
  if constexpr (EXT) {
    // no parts were searched: with one mismatch at most, every gapped
    // alignment scores less than both of the diagonal's ends
    if (one && mism <= 1) {
      const int full = sa * m - (mism ? sa - sb : 0);
      // the early end is before the mismatch or at the read's end
      const int before = mism ? hit[0] : m;
      const int early = sa * before >= full ? before : m;
      const int escore = h0 + (early == m ? full : sa * early);
      direct = sa * m - full < gap;
      const bool whole = (long)h0 + full >= (long)escore - (long)prm->ext_clip;
      score = whole ? h0 + full : escore;
      ie = whole ? m : early;
    }
  } else {
    bool leaves = false;  // leaving the diagonal might pay
    const int lose2 = 2 * (sa - sb);
    const int cx2 = LOCAL ? prm->pr_costs.leave2_local : prm->pr_costs.leave2;
    const int few = known ? mism : 0;
    auto saved2 = [&](int from, int to, int k, int free) -> int {
      return leave_saves2(lose2, cx2, T, from, to, k, free);
    };
    for (int i = x; i < few; i += 8) {
      const int pi = hit[i];
      int head = saved2(0, pi, i + 1, LOCAL ? 2 : 1), tail = saved2(pi, m - 1, mism - i, LOCAL ? 2 : 1);
      if constexpr (LOCAL) {  // clipping the stretch loses no more than a per base
        head = head < 2 * sa * (pi + 1) ? head : 2 * sa * (pi + 1);
        tail = tail < 2 * sa * (m - pi) ? tail : 2 * sa * (m - pi);
      }
      leaves |= head >= 2 * gap || tail >= 2 * gap;
      for (int j = i; j < few; ++j) leaves |= saved2(pi, hit[j], j - i + 1, 2) >= 4 * gap;
    }
    leaves = (__ballot(leaves) >> (8 * q) & 0xFFu) != 0;
    if (busy) {
      int at = 0;  // mismatches of the first and (from bit 16) of the last part
      for (int i = x; i < few; i += 8) at += (hit[i] < kSeed ? 1 : 0) + (hit[i] >= m - kSeed ? 0x10000 : 0);
      at = sum8(at);
      crowd = (at & 0xFFFF) > (at >> 16) ? at & 0xFFFF : at >> 16;
    }
    if (known && (busy || !leaves)) {
      if constexpr (LOCAL) {
        // the best stretch of the diagonal: H along it, back to 0 where it
        // would not stay above (the traceback stops at the last 0)
        int hcur = 0, from = 0, at = 0;
        for (int j = 0; j <= few; ++j) {
          const int to = j < few ? hit[j] : m;
          hcur += sa * (to - at);
          if (hcur > score) {
            score = hcur;
            ie = to;
            i0 = from;
          }
          hcur += sb;
          if (hcur <= 0) {
            hcur = 0;
            from = to + 1;
          }
          at = to + 1;
        }
      } else {
        score = sa * m - (sa - sb) * mism;
        ie = m;
      }
      direct = !leaves && loss_certain(prm->pr_costs, LOCAL, T, sa * m - score);
    }
  }
  // (ie = 0: the anchor itself, or a local read that matches nowhere)
  direct = direct && ie > 0;
  if (!SAMPLE && direct && x == 0) {
    const int je = ie + c0;
    G(prm->score)[p] = score;
    G(prm->read_end)[p] = ie;
    G(prm->ref_end)[p] = je;
    uint32_t st = 0;
    if constexpr (TRACE) {
      G(prm->read_start)[p] = i0;
      G(prm->ref_start)[p] = i0 + c0;
      if (prm->flags & kOutCigar) {
        if (prm->cigar_cap >= 1) {
          G(prm->cigar)[(size_t)p * (size_t)prm->cigar_cap] = (uint32_t)(ie - i0) << 4;
          G(prm->n_cigar)[p] = 1;
        } else {
          st = kStCigarTrunc;
          G(prm->n_cigar)[p] = -1;
        }
      }
      band_count<V, MODE>(prm, m, n, h0, score, ie, je, count);
    }
    G(prm->status)[p] = st;
  }

  // ---- the band the others need ------------------------------------------------
  int ns = 0, lo = 0, margin = 0;
  if (ok && !direct) {
    if constexpr (EXT) {
      const long loss = (long)h0 + (long)sa * m - best + prm->ext_clip;
      const int lc = loss > (1 << 20) ? 1 << 20 : (int)loss;
      const int xd = loss_drift(prm->pr_costs, core, lc);
      const int xi = lc >= so + sa + se ? (lc - so) / (sa + se) : 0;
      lo = -(xi < m ? xi : m);
      const int hi = xd < n ? xd : n;
      ns = (hi - lo + 16) >> 4;
      margin = kProven;
    } else {
      // the loss to expect.  Of an alignment along the one diagonal, its own,
      // which bounds the best one's, so a band for it is certain to hold; a gap
      // (a word full of mismatches) may lose less.  Else u of T parts without an
      // occurrence hold T ln(T / (T - u)) substitutions where they fall at
      // random.  (With one for each part, 70% of reads of 100 bases with 10%
      // errors went to a band, three quarters of them for nothing: 100,000 in
      // windows of 214: 705 us of bands in place of 194.)  Where a band that fails
      // is cheap beside a pair left, one substitution a part is hoped for.
      auto subs = [&](int u) -> int {
        if (u < 1) return 0;
        if (!busy) return (sa - sb) * u;
        const float f = (float)u * __builtin_amdgcn_rcpf((float)T);
        return (sa - sb) * (int)((float)u * (1.0f + f * (0.5f + f * 0.3333f)));
      };
      int loss;
      bool sure = false;  // an alignment of this loss is known
      if (core.span > 0) {
        loss = so + (se + sa) * (core.span < 4 ? core.span : 4) + subs(missed - 1);
      } else if (one) {
        loss = score > 0 ? sa * m - score : (sa - sb) * total;
        sure = true;
        // (or one next to an end: three mismatches of its last bases)
        int other = crowd >= 3 ? so + 2 * se + (sa - sb) * (total - crowd) : loss;
        if (dense > 0) {
          const int gap = so + 2 * se + (sa - sb) * (total - dense + 1);
          other = gap < other ? gap : other;
          if constexpr (LOCAL) {  // (or clipped)
            const int clip = 2 * sa * dense + (sa - sb) * (total - dense);
            other = clip < other ? clip : other;
          }
        }
        if (!busy) {
          const int hope = subs(missed) + (mism > missed + 1 ? so + 2 * se : 0);
          other = hope < other ? hope : other;
        }
        if (other < loss) {
          loss = other;
          sure = false;
        }
      } else {
        loss = so + 2 * se + subs(busy ? missed - 1 : missed);
      }
      ns = 99;
      // (scores alone: a band that fails costs more than it may save, and over 32
      // diagonals nearly as much as the table)
      if (loss_certain(prm->pr_costs, LOCAL, T, TRACE || sure ? loss : loss + loss / 4))
        ns = band_strips(core.span, loss_drift(prm->pr_costs, core, loss));
      if (!TRACE && ns > 2) ns = 99;
      margin = ns <= 4 ? band_margin(core.span, ns) : 0;
      lo = c0 - margin;
    }
  }
  // (a band's cell costs some four of the table's: wide bands of short extensions
  // more than their scores; not more than a traceback, where a few pairs left
  // take the time of a whole round of items)
  if (EXT && !TRACE && busy && (ns > 2 ? 512 : 256) > 3 * n) ns = 99;
  const bool go = ok && !direct && ns <= 4;
  if constexpr (!SAMPLE) {
    if (go && x == 0) {
      G(prm->bucket_of)[p] = band_word(lo, margin, ns > 1 ? ns : 1);
      G(prm->dbsorted)[p] = core_word(core);
    }
    put_out(lds, 0, &cnt[0], valid && x == 0 && !direct && !go, (uint32_t)p);
    put_out(lds, 1, &cnt[1], x == 0 && go && ns <= 1, (uint32_t)p);
    put_out(lds, 2, &cnt[2], x == 0 && go && ns == 2, (uint32_t)p);
    put_out(lds, 3, &cnt[3], x == 0 && go && ns > 2, (uint32_t)p);
  }
  lds_wait();
  if constexpr (SAMPLE) {
    int v = 0;
    if (valid && x == 0) {
      v = -(1400 + m * n / 20);
      if (direct || go) v += TRACE ? m * (n + 64) / 10 * (LOCAL ? 15 : 11) : m * n;
      if (go) v -= m * (TRACE ? 112 : 90) * (ns > 2 ? 4 : (ns > 1 ? 2 : 1));
    }
#pragma unroll
    for (int s = 8; s < 64; s <<= 1) v += __shfl_xor(v, s, 64);
    *saved = v;  // of lane 0
  }
  return __builtin_popcountll(__ballot(x == 0 && (direct || go)));
}

// Block 0: the planner's scan.  The others look at a sample of the batch,
// kSampleWaves items of 8 pairs spread over it, so that the scan below is spared
// a batch without hope: what it finds of unrelated pairs, or of reads with too
// many errors for a certificate, does not pay for its looking (100,000 local
// reads of 60 in windows of 154, 5% errors, traced: 761 us with the scan, 677
// without).  An item's time (10-20 us) in place of the 5 of block 0 alone.
template <class V, bool TRACE>
__global__ __launch_bounds__(kScanThreads) void k_seed_sample(const Params* __restrict__ prm) {
  constexpr int KIND = V::kPairs == 1 ? kK32 : kK16;
  extern __shared__ uint32_t smem[];
  static_assert(kScanTableWords <= kScanStaticWords, "the scan's tables fit a wave's LDS");
  if (blockIdx.x == 0) {
    scan_tables(prm, smem);
    return;
  }
  const int wave = uni((int)(threadIdx.x >> 6));
  if (wave >= prm->pr_sample_waves) return;
  const uint32_t w = (blockIdx.x - 1) * (uint32_t)prm->pr_sample_waves + (uint32_t)wave;
  const int q = (int)(threadIdx.x & 63) >> 3;
  const uint64_t at = (uint64_t)(w * kPruneItem + (uint32_t)q) * (uint64_t)prm->n_pairs / (kSampleWaves * kPruneItem);
  const int p = (int)at;
  const uint32_t b = G(prm->bucket_of)[p];
  const bool in = b != kSkip && bucket_kind((int)(b / kSubBins)) == KIND;
  const int md = in ? bucket_mode((int)(b / kSubBins)) : -1;
  uint32_t* lds = smem + wave * prm->pr_scan_words;
  BandCount count{0, 0};
  auto look = [&](auto mode) {
    constexpr int MODE = decltype(mode)::value;
    const uint64_t some = __ballot(md == MODE);
    if (some == 0) return;
    int saved = 0;
    const int got = prune_scan<V, MODE, TRACE, true>(prm, md == MODE, p, lds, nullptr, &count, &saved);
    if ((threadIdx.x & 63) == 0) {
      unsigned long long* const sum = (unsigned long long*)(prm->counters + kCtrSeed) + 2 * MODE;
      atomicAdd(sum, (unsigned long long)(__builtin_popcountll(some) >> 3) | (unsigned long long)got << 32);
      atomicAdd(sum + 1, (unsigned long long)(long long)saved);
    }
  };
  look(std::integral_constant<int, 0>{});
  look(std::integral_constant<int, 1>{});
  look(std::integral_constant<int, 2>{});
}

// Whether the sample says to leave a mode's pairs.  Beyond what k_seed_left
// takes in two rounds (three where few are left), the pairs left go through the
// fills and their side lists, whose time hardly falls below that of one round of items (300 us of 454
// for 100,000 traced pairs of 50 x 139, a quarter of which were left), so the
// saving has to be more than that: the lines that part 60 batches of 40,000 to
// 300,000 pairs best (most of those on the wrong side lose under 4%; 0.85 to
// 0.95 of the full tables' speed without them).
__host__ __device__ constexpr long long saved_cells(bool trace) { return trace ? 2000000000 : 1000000000; }
template <bool TRACE>
__device__ __forceinline__ bool hopeless(const Params* __restrict__ prm, int mode, int per) {
  const unsigned long long* const sum = (const unsigned long long*)(prm->counters + kCtrSeed) + 2 * mode;
  const uint32_t tried = (uint32_t)sum[0], found = (uint32_t)(sum[0] >> 32);
  const long long share = prm->n_pairs >> 10;
  if (8u * found < tried) return true;
  if (mode == 2 || tried == 0) return false;
  const long long left = (tried - found) * share, limit = (long long)per * prm->left_limit;
  if (TRACE && (2 * left <= limit || (4 * left <= 3 * limit && 4 * (tried - found) <= tried))) return false;
  return (long long)sum[1] * share < saved_cells(TRACE);
}

// The scan of every pair of the batch, pr_chunk items of 8 pairs per wave:
// their mode and class follow from the queue the planner laid out.
template <class V, bool TRACE>
__global__ __launch_bounds__(256, kScanWaves) void k_seed_scan(const Params* __restrict__ prm) {
  constexpr int KIND = V::kPairs == 1 ? kK32 : kK16;
  extern __shared__ uint32_t smem[];
  const int wave = uni((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const uint32_t w = blockIdx.x * (blockDim.x >> 6) + (uint32_t)wave;
  constexpr int P0 = prune_part(KIND, 0);
  const MICA_GLOBAL uint32_t* qs = G(prm->pqstart) + P0 * (kNumClasses + 1);
  const uint32_t total = qs[kNumModes * (kNumClasses + 1) - 1];
  const uint32_t chunk = (uint32_t)prm->pr_chunk;
  uint32_t it = qs[0] + w * chunk;
  const uint32_t end = it + chunk < total ? it + chunk : total;
  // lane: a mode's class position and its first item
  static_assert(kNumModes * kNumClasses <= 64, "a lane per mode and class");
  const bool in = lane < kNumModes * kNumClasses;
  const uint32_t starts = in ? qs[lane / kNumClasses * (kNumClasses + 1) + lane % kNumClasses] : 0xFFFFFFFFu;
  uint32_t* lds = smem + wave * prm->pr_scan_words;

  __shared__ int head[kWavesPerBlock][9];  // bucket, four counts, four list positions of each wave
  uint32_t leave = 0;                      // modes whose pairs pass unseen
  if (prm->pr_sampled)
    for (int md = 0; md < kNumModes; ++md) leave |= hopeless<TRACE>(prm, md, V::kPairs) ? 1u << md : 0u;
  BandCount count{0, 0};
  int cnt[4] = {0, 0, 0, 0};
  int mode = 0, bucket = -1;
  for (; it < end; ++it) {
    const int pos = __builtin_popcountll(__ballot(in && starts <= it)) - 1;
    const int md = pos / kNumClasses;
    const int b = bucket_id(KIND, prune_class(pos - md * kNumClasses), md);
    if (b != bucket && bucket >= 0) {
      // another bucket: what the wave has of this one goes by itself
      lds_wait();
      uint32_t at[4];
#pragma unroll
      for (int li = 0; li < 4; ++li) {
        at[li] = 0;
        if (lane == 0 && cnt[li]) at[li] = atomicAdd(out_count(prm, li, bucket), (uint32_t)cnt[li]);
        at[li] = wave_uniform(at[li]);
      }
      write_out<TRACE>(prm, mode, bucket, lds, cnt, at);
      cnt[0] = cnt[1] = cnt[2] = cnt[3] = 0;
      lds_wait();
    }
    mode = md;
    bucket = b;
    const uint32_t first = (it - (uint32_t)__builtin_amdgcn_readlane((int)starts, pos)) * kPruneItem;
    const uint32_t left = G(prm->bcount)[b] - first;
    const uint32_t* pairs = prm->presorted + G(prm->bstart)[b] + first;
    const int np = left < (uint32_t)kPruneItem ? (int)left : kPruneItem;
    if ((leave >> md) & 1u) {
      uint32_t p = 0;
      if (lane < np) p = G(pairs)[lane];
      put_out(lds, 0, &cnt[0], lane < np, p);
    } else {
      const bool valid = (lane >> 3) < np;
      const int p = valid ? (int)G(pairs)[lane >> 3] : 0;
      if (md == 0) prune_scan<V, 0, TRACE, false>(prm, valid, p, lds, cnt, &count);
      else if (md == 1) prune_scan<V, 1, TRACE, false>(prm, valid, p, lds, cnt, &count);
      else prune_scan<V, 2, TRACE, false>(prm, valid, p, lds, cnt, &count);
    }
  }

  // The block's waves ask for room together: the counts of a bucket serve
  // about one request in 12 ns, and a request per wave and list keeps them
  // busy for 75 us in 400,000 pairs.
  if (lane == 0) {
    head[wave][0] = bucket;
#pragma unroll
    for (int li = 0; li < 4; ++li) head[wave][1 + li] = cnt[li];
  }
  __syncthreads();
  int lead = wave;
  uint32_t at[4] = {0, 0, 0, 0};
  if (bucket >= 0) {
    uint32_t before = 0, sum = 0;  // of lane li's list
    for (int v = (int)(blockDim.x >> 6) - 1; v >= 0; --v) {
      if (head[v][0] != bucket) continue;
      uint32_t c = 0;
      if (lane < 4) c = (uint32_t)head[v][1 + lane];
      sum += c;
      if (v < wave) before += c;
      lead = v < lead ? v : lead;
    }
    if (lead == wave && lane < 4) head[wave][5 + lane] = sum ? (int)atomicAdd(out_count(prm, lane, bucket), sum) : 0;
#pragma unroll
    for (int li = 0; li < 4; ++li) at[li] = (uint32_t)__builtin_amdgcn_readlane((int)before, li);
  }
  __syncthreads();
  if (bucket >= 0) {
#pragma unroll
    for (int li = 0; li < 4; ++li) at[li] += (uint32_t)head[lead][5 + li];
    write_out<TRACE>(prm, mode, bucket, lds, cnt, at);
  }
  if constexpr (TRACE) band_count_flush(prm, count);
}

// A band item: the `take` pairs whose entries lie at the start of the wave's
// LDS, bands of up to LG diagonals, a group of LG lanes per packed couple.
// (A strip loop over 16-lane groups has a wide band's strips wait for each
// other: 0.46 us a row of three strips, 0.13 us in one wave-wide pass.)
template <class V, int MODE, bool TRACE, int LG>
__device__ __forceinline__ void prune_band(const Params* __restrict__ prm, int take, uint32_t* lds, uint8_t* slot,
                                           int* cnt, BandCount* count) {
  typedef typename V::T T;
  constexpr int NP = V::kPairs;
  constexpr bool LOCAL = (MODE == 1);
  constexpr bool EXT = (MODE == 2);
  constexpr bool TRACK = (MODE != 0);
  const int lane = threadIdx.x & 63;
  const int bg = lane / LG;
  const int l = lane & (LG - 1);
  MICA_GLOBAL uint32_t* rec = (MICA_GLOBAL uint32_t*)slot;
  BandFind<T, 1> find;
  {
    const MICA_GLOBAL uint32_t* __restrict__ ref2b = G(prm->ref2b);
    const MICA_GLOBAL uint32_t* __restrict__ reads2b = G(prm->reads2b);
    int mm[NP], nn[NP], dlo[NP], W[NP], d0[NP], h0[NP];
    uint64_t wo[NP], ro[NP];
    bool act[NP];
    int rows_l = 0, mr_l = 0, tail_l = -0x7FFFFFFF;
#pragma unroll
    for (int h = 0; h < NP; ++h) {
      const int q = bg * NP + h;
      act[h] = q < take;
      mm[h] = nn[h] = dlo[h] = d0[h] = h0[h] = 0;
      W[h] = 1;
      wo[h] = ro[h] = 0;
      if (act[h]) {
        const int p = (int)lds[q * kBandEntry];
        const uint32_t w1 = lds[q * kBandEntry + 1];
        mm[h] = G(prm->read_len)[p];
        nn[h] = G(prm->win_len)[p];
        wo[h] = G(prm->win_off)[p];
        ro[h] = G(prm->read_off)[p];
        if constexpr (EXT) h0[h] = prm->ext_h0 ? G(prm->ext_h0)[p] : prm->ext_default_h0;
        dlo[h] = (int)(w1 & 0xFFFFu) - 32768;
        W[h] = 16 * (int)(w1 >> 24);
        rows_l = mm[h] > rows_l ? mm[h] : rows_l;
      }
    }
    const int rows_u = wave_max_int(rows_l);
#pragma unroll
    for (int h = 0; h < NP; ++h) {
      // all pairs end on the wave's last row (extensions start on its first)
      const int top = !EXT && act[h] ? rows_u - mm[h] : 0;
      find.top[h] = top;
      if (dlo[h] < 0 && top - dlo[h] > mr_l) mr_l = top - dlo[h];
      dlo[h] -= top;
      if (!EXT) d0[h] = top;
      if (act[h]) {
        // the first row some diagonal of the pair has to be watched on
        int t = EXT ? mm[h] : rows_u + 1;
        if (TRACK) {
          const int e = nn[h] - (dlo[h] + W[h] - 1) + 1;
          t = e < t ? e : t;
        }
        tail_l = -t > tail_l ? -t : tail_l;
      }
    }
    const int mr_u = wave_max_int(mr_l);
    int tail_u = -wave_max_int(tail_l);
    tail_u = tail_u < 1 ? 1 : tail_u;

    // codes in LDS, as for the band refill, from the sequences' words, which
    // are all fetched at once (code by code from memory this took a third of
    // the band's time)
    uint32_t* gq = lds + kBandStaticWords + bg * prm->pr_group_words;
    uint16_t* gw = (uint16_t*)(gq + prm->pr_rows);
    uint32_t* const raw = lds + prm->pr_raw_off + bg * prm->pr_raw_words;
    const int rw = (rows_u + 15) >> 4, ww = (rows_u + LG + 15) >> 4;
    const uint64_t ref_last = (prm->ref_len - 1) >> 4, reads_last = (prm->reads_len - 1) >> 4;
#pragma unroll
    for (int h = 0; h < NP; ++h) {
      // read bases from row 0 on (dummy rows first), window columns from the
      // band's first on; positions outside read or window are never used
      uint32_t* const r = raw + h * (rw + ww);
      if (act[h]) {
        for (int w = l; w < rw; w += LG) {
          const int64_t at = (int64_t)ro[h] + 16 * w - find.top[h];
          r[w] = at + 15 >= 0 ? signed_word(reads2b, at, reads_last) : 0u;
        }
        for (int w = l; w < ww; w += LG) {
          const int64_t at = (int64_t)wo[h] + 16 * w + dlo[h] - 1;
          r[rw + w] = at + 15 >= 0 ? signed_word(ref2b, at, ref_last) : 0u;
        }
      }
    }
    lds_wait();
    for (int i0 = l; i0 < rows_u; i0 += LG) {
      uint32_t qs = 0;
#pragma unroll
      for (int h = 0; h < NP; ++h) {
        const uint32_t c = (raw[h * (rw + ww) + (i0 >> 4)] >> (2 * (i0 & 15))) & 3u;
        qs |= (act[h] && i0 >= find.top[h] && i0 - find.top[h] < mm[h]) ? V::qcode((int)c, h) : V::qdummy(h);
      }
      gq[i0] = qs;
    }
    const int ne = rows_u + LG;
    for (int e = l; e < ne; e += LG) {
      uint32_t w = 0;
#pragma unroll
      for (int h = 0; h < NP; ++h) {
        const int j = e + dlo[h];
        const uint32_t c = (raw[h * (rw + ww) + rw + (e >> 4)] >> (2 * (e & 15))) & 3u;
        if (act[h] && j >= 1 && j <= nn[h]) w |= c << (8 * h + (NP == 2 ? 1 : 0));
      }
      gw[e] = (uint16_t)w;
    }
    lds_wait();

    auto pack = [&](int v0, int v1) -> T {
      if constexpr (NP == 2) return V::make2(v0, v1);
      else return (T)v0;
    };
    find.m = pack(mm[0], mm[NP - 1]);
    find.best[0] = LOCAL ? pack(-d0[0], -d0[NP - 1]) : (T)V::kNeg;
    find.row[0] = (T)0;
    find.end[0] = (T)V::kNeg;
    int lim[2];
#pragma unroll
    for (int h = 0; h < NP; ++h) {
      const int e = nn[h] - (dlo[h] + l);
      lim[h] = EXT && mm[h] < e ? mm[h] : e;
    }
    find.lim[0] = pack(lim[0], lim[NP - 1]);
    band_refill<V, MODE, 1, TRACE, true, LG>(prm, dlo, W, d0, h0, act, rows_u, 1, mr_u, tail_u, gq, gw, rec, &find);
  }
  if constexpr (TRACE) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  lds_wait();
  if constexpr (TRACE) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

  // ---- result cell ---------------------------------------------------------------
  // The pairs' values are read again here (list, global arrays) rather than
  // kept across the rows.  The group's best: largest score, then smallest j,
  // then smallest i.
  constexpr int X = LG / NP;
  const int h_ = l / X;  // the pair this lane walks
  int p_ = 0, m_ = 0, n_ = 0, h0_ = 0, sc_ = 0, ie_ = 0, je_ = 0, dlo_ = 0, W_ = 0;
  uint32_t w1_ = 0, core_ = 0;
  int top_ = 0;
  bool act_ = false;
#pragma unroll
  for (int h = 0; h < NP; ++h) {
    const int q = bg * NP + h;
    const bool act = q < take;
    int p = 0, m = 0, n = 0, h0 = 0, dlo = 0, W = 0;
    uint32_t w1 = 0, cw = 0;
    if (act) {
      p = (int)lds[q * kBandEntry];
      w1 = lds[q * kBandEntry + 1];
      cw = lds[q * kBandEntry + 2];
      m = G(prm->read_len)[p];
      n = G(prm->win_len)[p];
      if constexpr (EXT) h0 = prm->ext_h0 ? G(prm->ext_h0)[p] : prm->ext_default_h0;
      dlo = (int)(w1 & 0xFFFFu) - 32768;
      W = 16 * (int)(w1 >> 24);
    }
    const int top = find.top[h];
    constexpr int kNone = -(1 << 28);  // below every score; its loss is certain of nothing
    int b0 = kNone, key0 = 0x7FFFFFFF;  // row m
    int b1 = kNone, key1 = 0x7FFFFFFF;  // any row
    const int dl = dlo + l;
    if (act && l < W) {
      if (!LOCAL) {
        const int j = m + dl;
        const int v = V::get(find.end[0], h) + top;
        if (j >= 0 && j <= n && v > b0) {
          b0 = v;
          key0 = j;
        }
      }
      if (TRACK) {
        const int v = V::get(find.best[0], h) + top;
        const int i = V::get(find.row[0], h) - top;
        if (i >= 1 && v > b1) {
          b1 = v;
          key1 = ((i + dl) << 11) | i;
        }
      }
    }
    auto reduce = [&](int b, int key, int* kout) -> int {
      int top = b;
#pragma unroll
      for (int d = 1; d < LG; d <<= 1) {
        const int o = __shfl_xor(top, d, 64);
        top = o > top ? o : top;
      }
      int k = b == top ? key : 0x7FFFFFFF;
#pragma unroll
      for (int d = 1; d < LG; d <<= 1) {
        const int o = __shfl_xor(k, d, 64);
        k = o < k ? o : k;
      }
      *kout = k;
      return top;
    };
    int k0 = 0, k1 = 0, sc, ie, je;
    if (!LOCAL) b0 = reduce(b0, key0, &k0);
    if (TRACK) b1 = reduce(b1, key1, &k1);
    if constexpr (MODE == 0) {
      sc = b0;
      ie = m;
      je = k0;
    } else {
      // the start cell (0, 0) is worth 0, or h0
      sc = h0;
      ie = je = 0;
      if (b1 > h0) {
        sc = b1;
        ie = k1 & 2047;
        je = k1 >> 11;
      }
      if (EXT && b0 != kNone && (long)b0 >= (long)sc - (long)prm->ext_clip) {
        sc = b0;
        ie = m;
        je = k0;
      }
    }
    if (h == 0 || h_ == h) {
      act_ = act;
      p_ = p;
      m_ = m;
      n_ = n;
      h0_ = h0;
      sc_ = sc;
      ie_ = ie;
      je_ = je;
      dlo_ = dlo;
      W_ = W;
      top_ = top;
      w1_ = w1;
      core_ = cw;
    }
  }

  // ---- is the band certain to hold every alignment this good? ------------------
  const bool lead = l == h_ * X;
  bool good = act_, again = false;
  int ns2 = 0, marg2 = 0;
  if (!EXT && act_) {
    const Core core = core_of(core_);
    const int margin = (int)((w1_ >> 16) & 0xFFu);
    const int loss = prm->sa * m_ - sc_;
    const bool sure = loss_certain(prm->pr_costs, LOCAL, m_ / kSeed, loss);
    const int drift = sure ? loss_drift(prm->pr_costs, core, loss) : 0;
    good = sure && drift <= margin;
    // a wider band will be (the loss can only shrink there)
    ns2 = band_strips(core.span, drift);
    again = sure && !good && ns2 <= 4;
    marg2 = band_margin(core.span, ns2);
    if (lead && again) w1_ = band_word(dlo_ + margin - marg2, marg2, ns2);
    if (lead && !good && !again) {
      const int bucket = bucket_id(NP == 1 ? kK32 : kK16, prm->class_of_m[m_], MODE);
      const uint32_t pos = atomicAdd(&prm->rcount[bucket], 1u);
      left_list<MODE, TRACE>(prm)[G(prm->bstart)[bucket] + pos] = (uint32_t)p_;
    }
  }
  if constexpr (!EXT) {
#pragma unroll
    for (int li = 0; li < 2; ++li) {
      const bool mine = lead && again && (ns2 <= 2) == (li == 0);
      const uint64_t bal = __ballot(mine);
      if (mine) {
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        uint32_t* e = lds + (kBandItem + li * kBandAgain + cnt[li] + (int)rank) * kBandEntry;
        e[0] = (uint32_t)p_;
        e[1] = w1_;
        e[2] = core_;
      }
      cnt[li] += __builtin_popcountll(bal);
    }
  }

  // ---- outputs ---------------------------------------------------------------------
  if (good) {
    if (lead) {
      G(prm->score)[p_] = sc_;
      G(prm->read_end)[p_] = ie_;
      G(prm->ref_end)[p_] = je_;
    }
    if constexpr (TRACE) {
      if (lead) band_count<V, MODE>(prm, m_, n_, h0_, sc_, ie_, je_, count);
      MICA_GLOBAL uint32_t* stg = (MICA_GLOBAL uint32_t*)(slot + prm->pr_rec_bytes) +
                                  (size_t)(bg * NP + h_) * (size_t)prm->stage_stride;
      band_walk<V, MODE, LG>(prm, rec, lds + kBandStaticWords + (bg * NP + h_) * kWalkStage, stg, 64, p_, m_, n_, ie_, je_, dlo_, W_, top_);
    } else {
      if (lead) G(prm->status)[p_] = 0;
    }
  }

  lds_wait();
}

// The full traceback of the pairs left, by whole waves of as few rows a lane
// as the item's reads need: those of up to 256 bases (LONG false) where they
// are few, at most four items per resident wave, so that the time of one item,
// which is then the launch's, is short (150 x 400: 3 rows a lane in place of 10, and
// of the 4 of the side lists' kernels, which also take a launch per mode and
// length range); longer ones always (their class has 16 rows a lane whatever
// the read).
template <class V, int MODE, bool LONG>
__device__ __forceinline__ void left_item(const Params* __restrict__ prm, const uint32_t* pairs, int np, int m,
                                          uint32_t* lds, uint8_t* slot, int bucket) {
  if constexpr (LONG) {
    if (m <= 384) process_item<V, 64, 6, MODE, kTbFull, false>(prm, pairs, np, lds, slot, bucket, nullptr, true);
    else if (m <= 512) process_item<V, 64, 8, MODE, kTbFull, false>(prm, pairs, np, lds, slot, bucket, nullptr, true);
    else if (m <= 768) process_item<V, 64, 12, MODE, kTbFull, false>(prm, pairs, np, lds, slot, bucket, nullptr, true);
    else process_item<V, 64, 16, MODE, kTbFull, false>(prm, pairs, np, lds, slot, bucket, nullptr, true);
  } else {
    if (m <= 128) process_item<V, 64, 2, MODE, kTbFull, false>(prm, pairs, np, lds, slot, bucket, nullptr, true);
    else if (m <= 192) process_item<V, 64, 3, MODE, kTbFull, false>(prm, pairs, np, lds, slot, bucket, nullptr, true);
    else process_item<V, 64, 4, MODE, kTbFull, false>(prm, pairs, np, lds, slot, bucket, nullptr, true);
  }
}
template <class V, int MODE, bool LONG>
__global__ __launch_bounds__(256, LONG ? 2 : 4) void k_seed_left(const Params* __restrict__ prm) {
  constexpr int KIND = V::kPairs == 1 ? kK32 : kK16;
  constexpr int PPI = V::kPairs;
  extern __shared__ uint32_t smem[];
  const int wave = uni((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int slot_id = (int)blockIdx.x * kWavesPerBlock + wave;
  if (slot_id >= prm->n_slots) return;
  // lane k: the class of position k, longest first
  const int c_ = prune_class(lane < kNumClasses ? lane : 0);
  const bool in = lane < kNumClasses && left_long(c_) == LONG;
  const uint32_t pairs = in ? G(prm->lcount)[bucket_id(KIND, c_, MODE)] : 0u;
  const uint32_t mine = (pairs + PPI - 1) / PPI;
  uint32_t upto = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(upto, d, 64);
    if (lane >= d) upto += o;
  }
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
  uint32_t* lds = smem + wave * kLdsWaveWords;
  uint8_t* slot = prm->scratch + (size_t)slot_id * prm->slot_bytes;
  for (uint32_t item = (uint32_t)slot_id; item < total; item += gridDim.x * (uint32_t)kWavesPerBlock) {
    const int k = __builtin_popcountll(__ballot(upto <= item));
    const uint32_t first = (item - ((uint32_t)__builtin_amdgcn_readlane((int)upto, k) -
                                    (uint32_t)__builtin_amdgcn_readlane((int)mine, k))) * PPI;
    const uint32_t have = (uint32_t)__builtin_amdgcn_readlane((int)pairs, k) - first;
    const int np = have < (uint32_t)PPI ? (int)have : PPI;
    const int bucket = bucket_id(KIND, prune_class(k), MODE);
    const uint32_t* list = (const uint32_t*)left_list<MODE, true>(prm) + G(prm->bstart)[bucket] + first;
    int m = 0;
    for (int s = 0; s < np; ++s) {
      const int ms = G(prm->read_len)[G(list)[s]];
      m = ms > m ? ms : m;
    }
    left_item<V, MODE, LONG>(prm, list, np, uni(m), lds, slot, bucket);
  }
}

// The bands of a mode, the wide ones first, in items of a wave's worth of
// pairs of one bucket.
template <class V, int MODE, bool TRACE>
__global__ __launch_bounds__(256, kBandWaves) void k_seed_band(const Params* __restrict__ prm) {
  constexpr int KIND = V::kPairs == 1 ? kK32 : kK16;
  constexpr int PART = prune_part(KIND, MODE);
  constexpr int P16 = 4 * V::kPairs, P32 = 2 * V::kPairs, P64 = V::kPairs;  // pairs per item
  extern __shared__ uint32_t smem[];
  const int wave = uni((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int waves = (int)(blockDim.x >> 6);
  const int slot_id = (int)blockIdx.x * waves + wave;
  if (slot_id >= prm->pr_slots) return;
  // lane k: class position k % kNumClasses of the list of up to 64 diagonals
  // (first), 32, 16
  static_assert(3 * kNumClasses <= 64, "a lane per class and list");
  uint32_t pairs = 0;
  const uint32_t ppi = lane < kNumClasses ? P64 : (lane < 2 * kNumClasses ? P32 : P16);
  if (lane < 3 * kNumClasses) {
    const int b = bucket_id(KIND, prune_class(lane % kNumClasses), MODE);
    const uint32_t* count_of = lane < kNumClasses ? prm->w64count : (lane < 2 * kNumClasses ? prm->w32count : prm->nbcount);
    pairs = G(count_of)[b];
  }
  const uint32_t mine = (pairs + ppi - 1) / ppi;
  uint32_t upto = mine;  // items of this lane and the ones before
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(upto, d, 64);
    if (lane >= d) upto += o;
  }
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
  if ((uint32_t)slot_id >= total) return;
  // wave k takes items k, k + waves, ...: the bands of a list cost nearly the
  // same, and a queue head serves only one request in 12 ns
  const uint32_t stride = (uint32_t)waves * gridDim.x < (uint32_t)prm->pr_slots ? (uint32_t)waves * gridDim.x
                                                                               : (uint32_t)prm->pr_slots;
  uint32_t* lds = smem + wave * prm->pr_band_words;
  uint8_t* slot = prm->scratch + (size_t)slot_id * prm->pr_slot_bytes;
  int cnt[2] = {0, 0};  // pairs to align again, with up to 32 and up to 64 diagonals
  BandCount count{0, 0};
  uint32_t item = (uint32_t)slot_id;
  for (;;) {
    const bool done = item >= total;
    // what to align next: pairs again, in a full item or at the end, or the
    // next item of the lists; its entries to the front of the LDS
    int width, take;
    const bool a32 = cnt[0] >= P32 || (done && cnt[0] > 0), a64 = cnt[1] >= P64 || (done && cnt[1] > 0);
    if (a32 || a64) {
      const int li = a32 ? 0 : 1;
      const int have = a32 ? cnt[0] : cnt[1];
      width = a32 ? 32 : 64;
      take = a32 ? (have < P32 ? have : P32) : (have < P64 ? have : P64);
      uint32_t* const own = lds + (kBandItem + li * kBandAgain) * kBandEntry;  // fewer than 64 words
      const uint32_t e = lane < have * kBandEntry ? own[lane] : 0u;
      lds_wait();
      if (lane < take * kBandEntry) lds[lane] = e;
      else if (lane < have * kBandEntry) own[lane - take * kBandEntry] = e;
      if (a32) cnt[0] -= take;
      else cnt[1] -= take;
    } else {
      if (done) break;
      const int k = __builtin_popcountll(__ballot(upto <= item));
      const int li = k / kNumClasses;  // 0: 64 diagonals, 1: 32, 2: 16
      width = li == 0 ? 64 : (li == 1 ? 32 : 16);
      const uint32_t per = li == 0 ? P64 : (li == 1 ? P32 : P16);
      const uint32_t first = (item - ((uint32_t)__builtin_amdgcn_readlane((int)upto, k) -
                                      (uint32_t)__builtin_amdgcn_readlane((int)mine, k))) * per;
      const uint32_t have = (uint32_t)__builtin_amdgcn_readlane((int)pairs, k) - first;
      take = (int)(have < per ? have : per);
      const int b = bucket_id(KIND, prune_class(k - li * kNumClasses), MODE);
      const uint32_t bs = G(prm->bstart)[b];
      const MICA_GLOBAL uint32_t* list =
          li == 0 ? G(prm->wlist) + bs + first
                  : band_list<MODE, TRACE>(prm) + (li == 1 ? bs + G(prm->bcount)[b] - first - (uint32_t)take : bs + first);
      if (lane < take) {
        const uint32_t p = list[lane];
        lds[lane * kBandEntry] = p;
        lds[lane * kBandEntry + 1] = G(prm->bucket_of)[p];
        lds[lane * kBandEntry + 2] = G(prm->dbsorted)[p];
      }
      item += stride;
    }
    lds_wait();
    if (width == 16) prune_band<V, MODE, TRACE, 16>(prm, take, lds, slot, cnt, &count);
    else if (width == 32) prune_band<V, MODE, TRACE, 32>(prm, take, lds, slot, cnt, &count);
    else prune_band<V, MODE, TRACE, 64>(prm, take, lds, slot, cnt, &count);
  }
  if constexpr (TRACE) band_count_flush(prm, count);
}

}  // namespace mica
