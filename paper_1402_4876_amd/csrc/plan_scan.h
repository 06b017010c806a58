// The planner's scan of the bucket table, run by one block (k_scan, k_front and
// the kernel that also samples the batch for the seeded bands).
#pragma once

#include "dp_common.h"

namespace mica {

// One block of kScanThreads, one thread per bucket and per queue position:
// bucket sizes and starts, the start of every (bucket, sub-bin) run inside
// its bucket, and the first work item of every queue position.
static_assert(kNumBuckets <= kScanThreads, "one thread per bucket");

// exclusive prefix sum over the block (within the waves by shuffles, their
// sums through sh); *total gets the sum
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* sh, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  uint32_t before = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) {
    const uint32_t x = sh[w];
    before += w < wave ? x : 0u;
    sum += x;
  }
  *total = sum;
  __syncthreads();
  return before + incl - v;
}

// (tab: kScanTableWords of LDS)
constexpr int kScanTableWords = kNumBuckets + kScanThreads;
__device__ __forceinline__ void scan_tables(const Params* __restrict__ prm, uint32_t* tab) {
  uint32_t* const cnt = tab;
  uint32_t* const sh = tab + kNumBuckets;
  const int b = threadIdx.x;
  uint32_t sub[kSubBins];
  uint32_t acc = 0;
  if (b < kNumBuckets) {
#pragma unroll
    for (int s = 0; s < kSubBins; ++s) {
      sub[s] = acc;
      acc += prm->scount[b * kSubBins + s];
    }
    cnt[b] = acc;
    prm->bcount[b] = acc;
  }
  uint32_t n_sorted;
  const uint32_t start = block_exclusive_scan(acc, sh, &n_sorted);  // also orders cnt[] before its reads
  // queue position q = b serves bucket qorder[q]
  uint32_t items = 0;
  if (b < kNumBuckets) {
    const int bq = (int)prm->qorder[b];
    const uint32_t ppi = (uint32_t)pairs_per_item(bucket_kind(bq), bucket_class(bq));
    items = (cnt[bq] + ppi - 1) / ppi;
  }
  uint32_t n_items;
  const uint32_t qs = block_exclusive_scan(items, sh, &n_items);
  if (b < kNumBuckets) {
    prm->qstart[b] = qs;
    prm->bstart[b] = start;
#pragma unroll
    for (int s = 0; s < kSubBins; ++s) prm->sfill[b * kSubBins + s] = start + sub[s];
  }
  if (prm->presorted) {
    // the band kernels' queue: thread = (part, class position)
    const int part = b / kNumClasses, pos = b - part * kNumClasses;
    const bool in = part < kPruneParts;
    uint32_t pi = 0;
    if (in) {
      const int bq = bucket_id(part < kNumModes ? kK16 : kK32, prune_class(pos), part % kNumModes);
      pi = (cnt[bq] + kPruneItem - 1) / kPruneItem;
    }
    uint32_t all;
    const uint32_t ps = block_exclusive_scan(pi, sh, &all);
    if (in) {
      prm->pqstart[part * (kNumClasses + 1) + pos] = ps;
      if (pos == kNumClasses - 1) prm->pqstart[part * (kNumClasses + 1) + kNumClasses] = ps + pi;
    }
    if (b < kNumBuckets) {
      prm->rcount[b] = prune_kind(bucket_kind(b)) ? 0u : acc;
      prm->nbcount[b] = 0;
      prm->w32count[b] = 0;
      prm->w64count[b] = 0;
    }
  }
  if (b == 0) {
    prm->qstart[kNumBuckets] = n_items;
    prm->counters[kCtrItems] = n_items;
    for (int q = 0; q < kPersistParts; ++q) prm->counters[kCtrQueueHead + q] = 0;
    prm->counters[kCtrRerun] = 0;
  }
  (void)n_sorted;
}

}  // namespace mica
