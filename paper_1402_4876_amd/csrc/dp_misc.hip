// Planning, bucketing, 2-bit packing and saturated-pair re-run kernels, and
// the table of kernel entry points used by the host runtime.
#include "dp_fill.h"
#include "plan.h"
#include "plan_scan.h"

namespace mica {

// Exact 32-bit recomputation of the pairs whose 16-bit scores saturated.
template <bool DIR>
__global__ __launch_bounds__(256) void k_rerun(const Params* __restrict__ prm) {
  extern __shared__ uint32_t smem[];
  const int wave = uni((int)(threadIdx.x >> 6));
  const int slot_id = blockIdx.x * kWavesPerBlock + wave;
  if (slot_id >= prm->n_slots) return;
  uint32_t* lds = smem + wave * kLdsWaveWords;
  uint8_t* slot = prm->scratch + (size_t)slot_id * prm->slot_bytes;
  const uint32_t cnt = prm->counters[kCtrRerun];
  const uint32_t n_waves = gridDim.x * (uint32_t)kWavesPerBlock;
  for (uint32_t it = (uint32_t)slot_id; it < cnt; it += n_waves) {
    const uint32_t* pp = prm->rerun + it;
    const int p = (int)*pp;
    const int md = prm->mode ? prm->mode[p] : prm->default_mode;
    // a full traceback: the re-run is rare and needs no band
    constexpr int TB = DIR ? kTbFull : kTbNone;
    if (md == 2) process_item<V32, 64, 16, 2, TB, false>(prm, pp, 1, lds, slot, -1);
    else if (md == 1) process_item<V32, 64, 16, 1, TB, false>(prm, pp, 1, lds, slot, -1);
    else process_item<V32, 64, 16, 0, TB, false>(prm, pp, 1, lds, slot, -1);
    if ((threadIdx.x & 63) == 0) prm->status[p] |= kStSaturated;
  }
}

// ----------------------------------------------------------------------------
// planning: validation, trivial pairs, bucket histogram, work queue

__device__ __forceinline__ void zero_tables(const Params* __restrict__ prm) {
  for (int i = threadIdx.x; i < kNumSubBuckets; i += blockDim.x) prm->scount[i] = 0;
  const int i = threadIdx.x;
  if (i < kNumBuckets) {
    prm->bhead[i] = 0;
    prm->fbcount[i] = 0;
    prm->dbcount[i] = 0;
    prm->dbwide[i] = 0;
    prm->sidehead[i] = 0;
  }
  if (i < kNumCounters) prm->counters[i] = 0;
}

__global__ void k_zero(const Params* __restrict__ prm) { zero_tables(prm); }

// Can every value of the pair's DP stay inside int16 (with a guard band)?
// Semi-global and local values are shifted by -d0 (dummy rows above the
// read).  An extension starts from h0: no cell exceeds h0 + a min(m, n),
// and every cell is at least what the path of j deletions along row 0 and i
// insertions down column j gives, h0 - 2o - (i + j)e, so every H, gap and
// boundary value is at least h0 - 3o - (m + n + 1)e.  (Rows below the read
// only feed rows further below; their values may clamp.)
__device__ __forceinline__ bool int16_safe(int m, int n, int mode, int d0, int a, int b, int o, int e, int h0) {
  long hi, lo;
  if (mode == 2) {
    hi = (long)h0 + (long)a * (long)(m < n ? m : n);
    lo = (long)h0 - 3L * o - (long)(m + n + 1) * e;
  } else {
    hi = (long)a * (long)(m < n ? m : n) - d0;
    lo = (mode ? -(long)(o + e) : -(long)(2 * o + (long)(m + 1) * e)) - d0;
  }
  (void)b;
  return hi <= 32767 - 8 && lo >= -32767 + 8;
}

// One pair: validation, and the result at once where there is nothing to
// align; else its bucket and length bin (counted in hist), kSkip otherwise.
__device__ __forceinline__ uint32_t plan_pair(const Params* __restrict__ prm, int64_t p, uint32_t* hist) {
  const int m = prm->read_len[p], n = prm->win_len[p];
  const int md = prm->mode ? (int)prm->mode[p] : prm->default_mode;
  const uint64_t wo = prm->win_off[p], ro = prm->read_off[p];
  const int h0 = md == 2 ? (prm->ext_h0 ? prm->ext_h0[p] : prm->ext_default_h0) : 0;
  uint32_t st = 0;
  if (m < prm->min_m || n < 0 || m > prm->max_m || n > prm->max_n || md < 0 || md > 2 || !((prm->mode_mask >> md) & 1) ||
      h0 < 0 || h0 > prm->max_h0)
    st = kStLenLimit;
  else if (wo > prm->ref_len || (uint64_t)n > prm->ref_len - wo) st = kStWinOob;
  else if (ro > prm->reads_len || (uint64_t)m > prm->reads_len - ro) st = kStReadOob;
  const bool want_start = (prm->flags & (kOutStart | kOutCigar)) != 0;
  const bool want_cigar = (prm->flags & kOutCigar) != 0;
  uint32_t b = kSkip;
  if (st != 0 || m == 0 || n == 0) {
    int score = 0, re = 0;
    int ncig = 0;
    // semi-global against an empty window: all insertions; an extension
    // with an empty read or window: the anchor itself, or (empty window)
    // all insertions when that is within the clipping penalty
    const bool all_ins = st == 0 && m > 0 &&
                         (md == 0 || (md == 2 && (long)prm->so + (long)m * prm->se <= (long)prm->ext_clip));
    if (st == 0 && md == 2) score = h0;
    if (all_ins) {
      score = (md == 2 ? h0 : 0) - (prm->so + m * prm->se);
      re = m;
      ncig = 1;
      if (want_cigar) {
        if (prm->cigar_cap >= 1) prm->cigar[(size_t)p * prm->cigar_cap] = ((uint32_t)m << 4) | 1u;
        else st |= kStCigarTrunc;
      }
    }
    prm->score[p] = score;
    prm->read_end[p] = re;
    prm->ref_end[p] = 0;
    if (want_start) {
      prm->read_start[p] = 0;
      prm->ref_start[p] = 0;
    }
    if (want_cigar) prm->n_cigar[p] = (st & kStCigarTrunc) ? -ncig : ncig;
    prm->status[p] = st;
  } else {
    const int cls = prm->class_of_m[m];
    const int d0 = class_lanes(cls) * class_rows(cls) - m;
    // the 16-bit bounds hold for the fallback class's dummy rows too
    // (at least as many as the pair's own class)
    const int fbc = fallback_class(cls);
    const int d0k = class_lanes(fbc) * class_rows(fbc) - m;
    int kind;
    if (prm->flags & kForceInt32) kind = kK32;
    else kind = int16_safe(m, n, md, d0k, prm->sa, prm->sb, prm->so, prm->se, h0) ? kK16 : kK16Sat;
    b = (uint32_t)(bucket_id(kind, cls, md) * kSubBins + sub_bin(cls, d0));
    atomicAdd(&hist[b], 1u);
  }
  prm->bucket_of[p] = b;
  return b;
}

__global__ __launch_bounds__(kPlanThreads) void k_plan(const Params* __restrict__ prm) {
  __shared__ uint32_t hist[kNumSubBuckets];
  for (int i = threadIdx.x; i < kNumSubBuckets; i += blockDim.x) hist[i] = 0;
  __syncthreads();
  for (int rep = 0; rep < kPlanPairsPerThread; ++rep) {
    const int64_t p = ((int64_t)blockIdx.x * kPlanPairsPerThread + rep) * blockDim.x + threadIdx.x;
    if (p < prm->n_pairs) (void)plan_pair(prm, p, hist);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kNumSubBuckets; i += blockDim.x)
    if (hist[i]) atomicAdd(&prm->scount[i], hist[i]);
}

__global__ __launch_bounds__(kScanThreads) void k_scan(const Params* __restrict__ prm) {
  __shared__ uint32_t tab[kScanTableWords];
  scan_tables(prm, tab);
}

// After the banded fills: the first work item of every queue position of
// the persistent buckets in the two side lists of the fills (fb: bands too
// wide for the refill; db: bands of 17-64 diagonals).
__device__ __forceinline__ void sidescan_tables(const Params* __restrict__ prm, uint32_t* sh) {
  const int q = threadIdx.x;
#pragma unroll 1
  for (int list = 0; list < 2; ++list) {
    uint32_t* qstart = list ? prm->dbqstart : prm->fbqstart;
    uint32_t items = 0;
    if (q < kNumBuckets) {
      const int b = (int)prm->qorder[q];
      if (persistent_bucket(b)) {
        const int cls = list ? bucket_class(b) : fallback_class(bucket_class(b));
        const uint32_t ppi = (uint32_t)pairs_per_item(bucket_kind(b), cls);
        items = list ? (prm->dbwide[b] + ppi - 1) / ppi + (prm->dbcount[b] + ppi - 1) / ppi
                     : (prm->fbcount[b] + ppi - 1) / ppi;
      }
    }
    uint32_t total;
    const uint32_t qs = block_exclusive_scan(items, sh, &total);
    if (q < kNumBuckets) qstart[q] = qs;
    if (q == 0) qstart[kNumBuckets] = total;
    __syncthreads();
  }
}

__global__ __launch_bounds__(kScanThreads) void k_sidescan(const Params* __restrict__ prm) {
  __shared__ uint32_t sh[kScanThreads];
  sidescan_tables(prm, sh);
}

// After the band kernels: the pairs they left, to k_seed_left, to the full
// traceback of the side lists or to the fills.
__global__ __launch_bounds__(kScanThreads) void k_rescan(const Params* __restrict__ prm) {
  __shared__ uint32_t sh[kScanThreads];
  const int q = threadIdx.x;
  const bool traced = (prm->flags & (kOutStart | kOutCigar)) != 0;
  auto seeded = [&](int b) { return traced && prune_kind(bucket_kind(b)); };
  // short reads: few enough for the kernel that takes them a wave an item?
  uint32_t waves = 0, all_waves;
  if (q < kNumBuckets && seeded(q) && !left_long(bucket_class(q))) {
    const uint32_t per = bucket_kind(q) == kK32 ? 1u : 2u;
    waves = (prm->rcount[q] + per - 1) / per;
  }
  (void)block_exclusive_scan(waves, sh, &all_waves);
  const bool few = all_waves <= (uint32_t)prm->left_limit;
  auto by_wave = [&](int b) { return seeded(b) && (few || left_long(bucket_class(b))); };
  auto full = [&](int b) { return seeded(b) && !by_wave(b) && left_full(prm, bucket_mode(b)); };
  uint32_t items = 0, left = 0;
  if (q < kNumBuckets) {
    const int bq = (int)prm->qorder[q];
    const uint32_t ppi = (uint32_t)pairs_per_item(bucket_kind(bq), bucket_class(bq));
    items = by_wave(bq) || full(bq) ? 0u : (prm->rcount[bq] + ppi - 1) / ppi;
    left = full(q) ? prm->rcount[q] : 0u;
    prm->lcount[q] = by_wave(q) ? prm->rcount[q] : 0u;
    prm->bcount[q] = by_wave(q) || full(q) ? 0u : prm->rcount[q];
    prm->fbcount[q] = left;
  }
  uint32_t n_items, n_left;
  const uint32_t qs = block_exclusive_scan(items, sh, &n_items);
  (void)block_exclusive_scan(left, sh, &n_left);
  if (q < kNumBuckets) prm->qstart[q] = qs;
  if (q == 0) {
    prm->qstart[kNumBuckets] = n_items;
    prm->counters[kCtrItems] = n_items;
    prm->counters[kCtrPruneLeft] = n_left;
  }
  // (a batch without extensions has no fill between here and the side lists)
  __syncthreads();
  __threadfence_block();
  sidescan_tables(prm, sh);
}

__global__ __launch_bounds__(kPlanThreads) void k_scatter(const Params* __restrict__ prm) {
  __shared__ uint32_t cnt[kNumSubBuckets];
  __shared__ uint32_t base[kNumSubBuckets];
  for (int i = threadIdx.x; i < kNumSubBuckets; i += blockDim.x) cnt[i] = 0;
  __syncthreads();
  uint32_t b[kPlanPairsPerThread], rank[kPlanPairsPerThread];
#pragma unroll
  for (int rep = 0; rep < kPlanPairsPerThread; ++rep) {
    const int64_t p = ((int64_t)blockIdx.x * kPlanPairsPerThread + rep) * blockDim.x + threadIdx.x;
    b[rep] = kSkip;
    rank[rep] = 0;
    if (p < prm->n_pairs) {
      b[rep] = prm->bucket_of[p];
      if (b[rep] != kSkip) rank[rep] = atomicAdd(&cnt[b[rep]], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kNumSubBuckets; i += blockDim.x)
    base[i] = cnt[i] ? atomicAdd(&prm->sfill[i], cnt[i]) : 0;
  __syncthreads();
#pragma unroll
  for (int rep = 0; rep < kPlanPairsPerThread; ++rep) {
    const int64_t p = ((int64_t)blockIdx.x * kPlanPairsPerThread + rep) * blockDim.x + threadIdx.x;
    if (b[rep] != kSkip) {
      uint32_t* to = prm->presorted && prune_kind(bucket_kind((int)b[rep] / kSubBins)) ? prm->presorted : prm->sorted;
      to[base[b[rep]] + rank[rep]] = (uint32_t)p;
    }
  }
}

// A small batch (at most kFrontPairs pairs): clearing, planning, scans and
// scatter in one block, in place of four launches (each some 5 us of start
// and drain for less than 1 us of work).
__global__ __launch_bounds__(kScanThreads) void k_front(const Params* __restrict__ prm) {
  __shared__ uint32_t hist[kNumSubBuckets];
  __shared__ uint32_t tab[kScanTableWords];
  const int n = (int)prm->n_pairs;
  zero_tables(prm);
  for (int i = threadIdx.x; i < kNumSubBuckets; i += kScanThreads) hist[i] = 0;
  __syncthreads();
  for (int p = threadIdx.x; p < n; p += kScanThreads) (void)plan_pair(prm, p, hist);
  __syncthreads();
  for (int i = threadIdx.x; i < kNumSubBuckets; i += kScanThreads) prm->scount[i] = hist[i];
  __threadfence();
  __syncthreads();
  scan_tables(prm, tab);
  __threadfence();
  __syncthreads();
  for (int i = threadIdx.x; i < kNumSubBuckets; i += kScanThreads)
    if (hist[i]) hist[i] = prm->sfill[i];
  __syncthreads();
  for (int p = threadIdx.x; p < n; p += kScanThreads) {
    const uint32_t b = prm->bucket_of[p];
    if (b == kSkip) continue;
    uint32_t* to = prm->presorted && prune_kind(bucket_kind((int)b / kSubBins)) ? prm->presorted : prm->sorted;
    to[atomicAdd(&hist[b], 1u)] = (uint32_t)p;
  }
}

// A lane packs kPackWords words, a block's stride apart, from 16 codes each.
// Bound by memory: one 16-byte load a word where the codes are aligned for it,
// as those of an allocation are (30.3 MB: 11.8 us, the launch
// included; 16 byte loads for the one word of a lane took 34.7 us), single bytes elsewhere and for the last word.
constexpr int kPackWords = 4;
__global__ __launch_bounds__(256) void k_pack2bit(const uint8_t* __restrict__ codes, int64_t n,
                                                   uint32_t* __restrict__ words) {
  const int64_t nw = (n + 15) / 16;
  const int64_t w0 = (int64_t)blockIdx.x * (kPackWords * 256) + threadIdx.x;
  if (((uintptr_t)codes & 15u) == 0 && ((int64_t)blockIdx.x + 1) * (kPackWords * 256) * 16 <= n) {
    uint4 c[kPackWords];
#pragma unroll
    for (int u = 0; u < kPackWords; ++u) c[u] = *(const uint4*)(codes + (w0 + u * 256) * 16);
    auto four = [](uint32_t x) -> uint32_t {
      x &= 0x03030303u;
      return (x | (x >> 6) | (x >> 12) | (x >> 18)) & 0xFFu;
    };
#pragma unroll
    for (int u = 0; u < kPackWords; ++u)
      words[w0 + u * 256] = four(c[u].x) | (four(c[u].y) << 8) | (four(c[u].z) << 16) | (four(c[u].w) << 24);
    return;
  }
  for (int u = 0; u < kPackWords; ++u) {
    const int64_t w = w0 + u * 256;
    if (w >= nw) return;
    uint32_t v = 0;
    for (int x = 0; x < 16; ++x) {
      const int64_t i = w * 16 + x;
      if (i < n) v |= ((uint32_t)codes[i] & 3u) << (2 * x);
    }
    words[w] = v;
  }
}

}  // namespace mica

namespace mica {

// registration functions of the per-bucket fill kernels (one source file each)
#define MICA_FILL_DECL(kind, mode, dir) void reg_fill_##kind##_##mode##_##dir(KernelTable& t);
#define MICA_FILL_ALL(X) \
  X(k16, 0, 0) X(k16, 0, 1) X(k16, 1, 0) X(k16, 1, 1) \
  X(k16s, 0, 0) X(k16s, 0, 1) X(k16s, 1, 0) X(k16s, 1, 1) \
  X(k32, 0, 0) X(k32, 0, 1) X(k32, 1, 0) X(k32, 1, 1) \
  X(k16, 2, 0) X(k16, 2, 1) X(k16s, 2, 0) X(k16s, 2, 1) X(k32, 2, 0) X(k32, 2, 1)
MICA_FILL_ALL(MICA_FILL_DECL)
#define MICA_SIDE_ALL(X) X(k16, 0) X(k16, 1) X(k16, 2) X(k16s, 0) X(k16s, 1) X(k16s, 2) X(k32, 0) X(k32, 1) X(k32, 2)
#define MICA_SIDE_DECL(kind, mode) void reg_side_##kind##_##mode(KernelTable& t);
MICA_SIDE_ALL(MICA_SIDE_DECL)
#define MICA_PERSIST_ALL(X) \
  X(0, 0, 0) X(0, 0, 1) X(0, 1, 0) X(0, 1, 1) X(0, 2, 0) X(0, 2, 1) \
  X(1, 0, 0) X(1, 0, 1) X(1, 1, 0) X(1, 1, 1) X(1, 2, 0) X(1, 2, 1)
#define MICA_PERSIST_DECL(dir, mode, part) void reg_persistent_##dir##_##mode##_##part(KernelTable& t);
MICA_PERSIST_ALL(MICA_PERSIST_DECL)
#define MICA_PERSIST_SIDE_ALL(X) X(0, 0) X(0, 1) X(1, 0) X(1, 1) X(2, 0) X(2, 1)
#define MICA_PERSIST_SIDE_DECL(mode, part) void reg_persistent_side_##mode##_##part(KernelTable& t);
MICA_PERSIST_SIDE_ALL(MICA_PERSIST_SIDE_DECL)

#define MICA_SEED_ALL(X) \
  X(0, 0, 0) X(0, 0, 1) X(0, 0, 2) X(0, 1, 0) X(0, 1, 1) X(0, 1, 2) \
  X(1, 0, 0) X(1, 0, 1) X(1, 0, 2) X(1, 1, 0) X(1, 1, 1) X(1, 1, 2)
#define MICA_SEED_DECL(tb, wide, mode) void reg_seed_##tb##_##wide##_##mode(KernelTable& t);
MICA_SEED_ALL(MICA_SEED_DECL)

#define MICA_LEFT_ALL(X) \
  X(0, 0, 0) X(0, 0, 1) X(0, 1, 0) X(0, 1, 1) X(0, 2, 0) X(0, 2, 1) \
  X(1, 0, 0) X(1, 0, 1) X(1, 1, 0) X(1, 1, 1) X(1, 2, 0) X(1, 2, 1)
#define MICA_LEFT_DECL(wide, mode, lng) void reg_seed_left_##wide##_##mode##_##lng(KernelTable& t);
#define MICA_LEFT_CALL(wide, mode, lng) reg_seed_left_##wide##_##mode##_##lng(*this);
MICA_LEFT_ALL(MICA_LEFT_DECL)

KernelTable::KernelTable() {
#define MICA_SEED_CALL(tb, wide, mode) reg_seed_##tb##_##wide##_##mode(*this);
  MICA_SEED_ALL(MICA_SEED_CALL)
  rescan = &k_rescan;
  MICA_LEFT_ALL(MICA_LEFT_CALL)
  front = &k_front;
#define MICA_FILL_CALL(kind, mode, dir) reg_fill_##kind##_##mode##_##dir(*this);
  MICA_FILL_ALL(MICA_FILL_CALL)
#define MICA_SIDE_CALL(kind, mode) reg_side_##kind##_##mode(*this);
  MICA_SIDE_ALL(MICA_SIDE_CALL)
#define MICA_PERSIST_CALL(dir, mode, part) reg_persistent_##dir##_##mode##_##part(*this);
  MICA_PERSIST_ALL(MICA_PERSIST_CALL)
#define MICA_PERSIST_SIDE_CALL(mode, part) reg_persistent_side_##mode##_##part(*this);
  MICA_PERSIST_SIDE_ALL(MICA_PERSIST_SIDE_CALL)
  sidescan = &k_sidescan;
  rerun[0] = &k_rerun<false>;
  rerun[1] = &k_rerun<true>;
  zero = &k_zero;
  plan = &k_plan;
  scan = &k_scan;
  scatter = &k_scatter;
}

const KernelTable& kernels() {
  static KernelTable t;
  return t;
}

hipError_t launch_pack2bit(const uint8_t* codes, int64_t n, uint32_t* words, hipStream_t s) {
  const int64_t nw = (n + 15) / 16;
  if (nw == 0) return hipSuccess;
  hipLaunchKernelGGL(k_pack2bit, dim3((unsigned)((nw + 256 * kPackWords - 1) / (256 * kPackWords))), dim3(256), 0, s, codes, n,
                     words);
  return hipGetLastError();
}

}  // namespace mica
