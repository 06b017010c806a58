// Internal definitions shared by the device kernels and the host runtime of
// the DP-phase library.  Nothing here is part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "seed_bound.h"

namespace mica {

constexpr int kMaxM = 1024;  // longest read (rows)
constexpr int kMaxN = 8192;  // longest window (columns)
constexpr int kMaxH0 = 1 << 20;  // largest extension anchor score and clipping penalty

// Kernel classes: class c < 16 runs 16 lanes per pair with c+1 read rows per
// lane (reads up to 16*(c+1) bases); classes 16, 17 and 18 run a whole wave
// (64 lanes) with 16, 4 and 8 rows per lane (reads up to 1024, 256 and 512
// bases).  The default plan uses classes 0-16; 17 and 18 are alternatives a
// tuned plan may pick.
constexpr int kNumClasses = 19;
__host__ __device__ constexpr int class_lanes(int c) { return c < 16 ? 16 : 64; }
__host__ __device__ constexpr int class_rows(int c) { return c < 16 ? c + 1 : (c == 16 ? 16 : (c == 17 ? 4 : 8)); }
// class of (lanes, rows), or -1
__host__ __device__ constexpr int class_of(int lanes, int rows) {
  return lanes == 16 ? (rows >= 1 && rows <= 16 ? rows - 1 : -1)
                     : (lanes == 64 ? (rows == 16 ? 16 : (rows == 4 ? 17 : (rows == 8 ? 18 : -1))) : -1);
}

// Arithmetic kinds: packed 16-bit (two pairs per 32-bit register), packed
// 16-bit with a run-time saturation check, and 32-bit.
enum Kind : int { kK16 = 0, kK16Sat = 1, kK32 = 2 };
constexpr int kNumKinds = 3;
// alignment modes: 0 semi-global, 1 local, 2 seed extension with clipping
constexpr int kNumModes = 3;
constexpr int kNumBuckets = kNumKinds * kNumClasses * kNumModes;
__host__ __device__ constexpr int bucket_id(int kind, int cls, int mode) {
  return (kind * kNumClasses + cls) * kNumModes + mode;
}
__host__ __device__ constexpr int bucket_kind(int b) { return b / (kNumModes * kNumClasses); }
__host__ __device__ constexpr int bucket_class(int b) { return (b / kNumModes) % kNumClasses; }
__host__ __device__ constexpr int bucket_mode(int b) { return b % kNumModes; }
// Within a bucket pairs are ordered by read length, longest first, in
// kSubBins bins of the dummy-row count d0 (one bin per row for the 16-lane
// classes, 16 rows per bin for the 64-lane ones, the last bin open-ended).
// A work item then holds reads of nearly equal length and, since windows
// usually grow with the read, nearly equal windows: its step count (the
// longest window of its pairs) wastes less on its shorter pairs, and the
// longest items of a bucket are taken first.
constexpr int kSubBins = 16;
constexpr int kNumSubBuckets = kNumBuckets * kSubBins;
__host__ __device__ constexpr int sub_bin(int cls, int d0) {
  return (class_lanes(cls) == 16 ? d0 : d0 >> 4) < kSubBins - 1 ? (class_lanes(cls) == 16 ? d0 : d0 >> 4)
                                                                 : kSubBins - 1;
}
// pairs handled by one wave-sized work item
__host__ __device__ constexpr int pairs_per_item(int kind, int cls) {
  return (kind == kK32 ? 1 : 2) * (64 / class_lanes(cls));
}
// The class whose kernels may trace a pair of class `cls` back in full when
// its band is too wide.  For the 16-lane classes of 8 rows or more it is the
// 64-lane class of 4 rows (256 row slots): a fourth of the rows per lane, so
// one such item, which runs alone at the end of a small batch, takes about
// a third of the time, for more work per pair (the extra dummy rows).  The
// persistent side-list kernels always use it; a per-bucket side launch uses
// it while its list is short against the resident waves.  (The planner
// checks the 16-bit bounds with this class's dummy rows.)
__host__ __device__ constexpr int fallback_class(int cls) {
  return class_lanes(cls) == 16 && class_rows(cls) >= 8 ? 17 : cls;
}
static_assert(class_lanes(17) == 64 && class_rows(17) == 4, "the 256-row class of 64 lanes");

// The persistent kernels serve the packed 16-bit buckets of the 16-lane
// classes (the bulk of short-read work), split in two class ranges per mode
// so that the short classes run with more resident waves: part 0 holds
// classes 0..kPersistSmallMax, part 1 the classes up to kPersistMaxClass.
// The other buckets run as plain per-bucket launches after them.
#ifndef MICA_PERSIST_MAX_CLASS
#define MICA_PERSIST_MAX_CLASS 15
#endif
constexpr int kPersistSmallMax = 9;
constexpr int kPersistMaxClass = MICA_PERSIST_MAX_CLASS;
__host__ __device__ constexpr bool persistent_bucket(int b) {
  return bucket_kind(b) == kK16 && class_lanes(bucket_class(b)) == 16 && bucket_class(b) <= kPersistMaxClass;
}
__host__ __device__ constexpr int persist_part(int cls) { return cls <= kPersistSmallMax ? 0 : 1; }
// queue part of a persistent (mode, part): the long-read part of a mode
// first (its items cost most), then the short-read part
__host__ __device__ constexpr int persist_queue_part(int mode, int part) { return mode * 2 + (part ? 0 : 1); }
constexpr int kPersistParts = 2 * kNumModes;
constexpr int kQueueParts = kPersistParts + 1;  // the persistent parts, then everything else
// the ordering key of buckets in the work queue
__host__ __device__ constexpr int queue_part(int b) {
  return persistent_bucket(b) ? persist_queue_part(bucket_mode(b), persist_part(bucket_class(b))) : kPersistParts;
}

constexpr uint32_t kSkip = 0xFFFFFFFFu;

// The seeded band kernels (seed.h) take the packed 16-bit and the 32-bit
// buckets, one kernel per kind and mode (a "prune part").  Their queue runs
// through a part's classes from the longest reads to the shortest, whatever
// the plan's lanes, so that neighbouring items hold reads of similar length.
static_assert(kMaxM / kSeed < 256, "a part's number fits beside its bases");
constexpr int kPruneParts = 2 * kNumModes;
constexpr int kPruneItem = 8;          // pairs per item of the scan
// Batches from this size on are sampled first (by so many waves, an item each),
// for scores alone or of reads below this length: a traced table of longer ones
// costs so much more than the scan that it pays for itself (100,000 of 150 x 400,
// all unrelated: 2.7 ms of 4.3; 10% errors: 2.4 of 3.9).
constexpr int kSamplePairs = 32768;
constexpr int kSampleRead = 128;
constexpr int kSampleWaves = 128;
static_assert(kSampleWaves * kPruneItem == 1024, "the batch is n_pairs / 1024 samples");
constexpr int kScanThreads = 256;      // one thread per bucket
constexpr int kScanChunk = 8;          // items a wave of the scan takes, at most
constexpr int kScanStaticWords = 192 + 4 * kPruneItem * kScanChunk;  // LDS words of a wave before its sequences (scan)
constexpr int kBandStaticWords = 128;   // and before its band codes (band)
__host__ __device__ constexpr int prune_part(int kind, int mode) { return (kind == kK32 ? kNumModes : 0) + mode; }
__host__ __device__ constexpr int prune_class(int pos) { return pos == 0 ? 16 : (pos == 1 ? 18 : (pos == 2 ? 17 : 18 - pos)); }
// classes whose left pairs k_seed_left takes always (else: while they are few)
__host__ __device__ constexpr bool left_long(int cls) { return class_lanes(cls) * class_rows(cls) > 256; }
__host__ __device__ constexpr bool prune_kind(int kind) { return kind != kK16Sat; }

// counters[] slots
// (queue heads of the persistent kernels: kCtrQueueHead + queue part)
// (queue heads of the persistent side-list kernels: kCtrSideHead + queue part)
enum : int {
  kCtrQueueHead = 0,
  kCtrRerun = kPersistParts,
  kCtrItems,
  kCtrRerunHead,
  kCtrSideHead,
  kCtrPruneWide = kCtrSideHead + kPersistParts,  // pairs the band kernels finished or left to the full
  kCtrPruneMid,                                 // traceback, by band width: over 64 diagonals, 17-64
  kCtrPruneLeft,                                // pairs left to the full traceback
  // per mode two 64-bit words of the sample: its pairs and, from bit 32, those that
  // would be answered or listed for a band; the cells this would save
  kCtrSeed = (kCtrPruneLeft + 2) / 2 * 2,
  kNumCounters = kCtrSeed + 4 * kNumModes
};

// per-pair status bits (same values as the public header)
constexpr uint32_t kStSaturated = 1u << 0;
constexpr uint32_t kStCigarTrunc = 1u << 1;
constexpr uint32_t kStLenLimit = 1u << 2;
constexpr uint32_t kStWinOob = 1u << 3;
constexpr uint32_t kStReadOob = 1u << 4;
constexpr uint32_t kStInternal = 1u << 5;

constexpr uint32_t kOutStart = 1u << 0;
constexpr uint32_t kOutCigar = 1u << 1;
constexpr uint32_t kForceInt32 = 1u << 8;

// LDS per wave (32-bit words): during the fill, a window-selector ring of 256
// columns for each of up to 4 lane groups; after it, the banded traceback's
// read and window codes in the same space.  The per-pair results (shifted score, i*, j*) and the
// extension's end-to-end candidates sit at the top.
constexpr int kRing = 256;
constexpr int kRingWords = 4 * kRing;
constexpr int kLdsWaveWords = 2048;
constexpr int kRedOff = kLdsWaveWords - 64;  // 8 pairs x 4 words
constexpr int kGslOff = kLdsWaveWords - 32;  // 8 pairs x 2 words
constexpr int kBandWords = kRedOff;          // band codes: [0, kRedOff)
static_assert(kRingWords <= kRedOff, "fill areas below the results");
constexpr int kWavesPerBlock = 4;
// widest band of the banded traceback (diagonals); wider pairs are traced
// back from a full fill of direction bits instead.  Bands up to
// kBandInlineW diagonals are refilled by the fill kernel (right after the
// fill, or in the 16-lane classes an item's worth at a time from the wave's
// pending list); wider ones by a later launch whose work items hold only
// such pairs.
constexpr int kBandMaxW = 64;
constexpr int kBandInlineW = 16;
// words at the end of a traceback slot that hold a wave's pending pairs
// (pairs whose band refill waits for an item's worth of them)
constexpr int kPendWords = 16;

struct Params {
  // batch (device pointers owned by the caller)
  const uint32_t* ref2b;
  uint64_t ref_len;
  const uint64_t* win_off;
  const int32_t* win_len;
  const uint32_t* reads2b;
  uint64_t reads_len;
  const uint64_t* read_off;
  const int32_t* read_len;
  const uint8_t* mode;
  int32_t default_mode;
  int32_t max_m, max_n;
  int32_t min_m;  // pairs with fewer read bases are rejected (a launch-planning bound)
  int64_t n_pairs;
  int32_t* score;
  int32_t* read_end;
  int32_t* ref_end;
  int32_t* read_start;
  int32_t* ref_start;
  uint32_t* cigar;
  int32_t cigar_cap;
  int32_t* n_cigar;
  uint32_t* status;
  int32_t sa, sb, so, se;  // match, mismatch, gap open, gap extend
  const int32_t* ext_h0;   // extension start score per pair (NULL: ext_default_h0)
  int32_t ext_default_h0;
  int32_t max_h0;          // largest extension start score accepted
  int32_t ext_clip;        // extension clipping penalty
  int32_t mode_mask;       // modes the batch may hold (bit per mode)
  uint32_t flags;
  // workspace (device memory of the context)
  uint32_t* bucket_of;         // [n_pairs] bucket * kSubBins + sub-bin, or kSkip
  uint32_t* sorted;            // [n_pairs] pair ids grouped by bucket, then sub-bin
  uint32_t* rerun;             // [n_pairs] pair ids to recompute with 32-bit scores
  uint32_t* bcount;            // [kNumBuckets]
  uint32_t* bstart;            // [kNumBuckets]
  uint32_t* scount;            // [kNumSubBuckets] pairs per (bucket, sub-bin)
  uint32_t* sfill;             // [kNumSubBuckets] next free position of each (bucket, sub-bin)
  uint32_t* qstart;            // [kNumBuckets + 1] first item of each queue position
  const uint32_t* qorder;      // [kNumBuckets] bucket served at each queue position
  const uint8_t* class_of_m;   // [kMaxM + 1]
  uint32_t* counters;          // [kNumCounters]
  uint32_t* bhead;             // [kNumBuckets] next work item of each plain bucket launch
  // The side lists of the banded fills: fb, pairs whose band was too wide
  // (full traceback); db, pairs with bands of 17-64 diagonals (refilled later)
  uint32_t* fbcount;           // [kNumBuckets] fb pairs per bucket
  uint32_t* fbsorted;          // [n_pairs] fb pairs, in their bucket's range of `sorted`
  uint32_t* fbqstart;          // [kNumBuckets + 1] first fb item of each queue position
  uint32_t* dbcount;           // [kNumBuckets] db pairs of 17-32 diagonals per bucket
  uint32_t* dbwide;            // [kNumBuckets] db pairs of 33-64 diagonals per bucket
  uint32_t* dbsorted;          // [n_pairs] db pairs in their bucket's range of `sorted`: 17-32
                               // diagonals from its start up, 33-64 from its end down
  uint32_t* dbqstart;          // [kNumBuckets + 1] first db item of each queue position
  uint32_t* sidehead;          // [kNumBuckets] next side-list item of each per-bucket side launch
  uint8_t* scratch;            // n_slots * slot_bytes
  uint64_t slot_bytes;         // per resident wave: direction bits + CIGAR staging
  uint64_t dir_bytes;          // direction-bit part of a slot
  int32_t stage_stride;        // CIGAR staging words per pair
  int32_t n_slots;             // resident waves the scratch is sized for
  // seeded band kernels (unused when presorted is NULL)
  uint32_t* presorted;         // [n_pairs] the planner's order; what they leave goes to `sorted`
  uint32_t* rcount;            // [kNumBuckets] pairs left per bucket
  uint32_t* lcount;            // [kNumBuckets] pairs left to k_seed_left
  int32_t left_full_;          // pairs left go to the full traceback without a fill (see left_full)
  int32_t left_limit;          // the items of short reads that k_seed_left takes
  int32_t pr_sampled;          // the batch has been sampled
  int32_t pr_sample_waves;     // waves a block that do so
  uint32_t* nbcount;           // [kNumBuckets] pairs on the band lists, of up to 16 diagonals
  uint32_t* w32count;          // [kNumBuckets] of 17-32
  uint32_t* w64count;          // [kNumBuckets] of 33-64
  uint32_t* wlist;             // [n_pairs] and the last of these lists, in the bucket's range
  uint32_t* pqstart;           // [kPruneParts][kNumClasses + 1] first queue item of each class
  uint64_t pr_slot_bytes, pr_rec_bytes;  // a wave's part of scratch, its band records
  int32_t pr_slots;
  int32_t pr_chunk;            // items per wave of the scan
  int32_t pr_scan_words, pr_band_words;  // LDS words per wave
  int32_t pr_win_words, pr_read_words, pr_part_words;  // scan: LDS words per pair
  int32_t pr_rows, pr_group_words;                     // band: rows, LDS words per group
  int32_t pr_raw_off, pr_raw_words;                    // and of its sequences
  SeedCosts pr_costs;          // what spoiling a read part costs
  uint32_t persist_q[kQueueParts];  // queue positions [persist_q[q], persist_q[q+1]) of queue part q
};

// Where many pairs are left of a batch with a traceback: to the full traceback
// at once, since most of them (unrelated, or far from their diagonal) would end
// there after a score-only fill too.  Not extensions and reads of up to 100
// bases, whose band is narrow more often than not.
__host__ __device__ inline bool left_full(const Params* p, int mode) { return p->left_full_ && mode != 2; }
constexpr int kLeftFullRead = 100;
// Reads below this are of few parts.
constexpr int kFewPartsRead = 72;

}  // namespace mica

namespace mica {
typedef void (*KernelFn)(const Params*);
// Kernel entry points of the library, indexed for the host runtime.
struct KernelTable {
  KernelFn bucket[2][kNumBuckets];  // [with traceback][bucket]
  KernelFn persistent[2][kNumModes][2];  // [with traceback][mode][class part]
  // the side lists after the banded fills: per bucket, and persistent over
  // the persistent buckets ([mode][class part]), after their item scan
  KernelFn side[kNumBuckets];
  KernelFn side_persistent[kNumModes][2];
  KernelFn sidescan;
  KernelFn seed_sample[2][2];           // [with traceback][32-bit]
  KernelFn seed_scan[2][2];
  KernelFn seed_band[2][2][kNumModes];  // [with traceback][32-bit][mode]
  KernelFn seed_left[2][kNumModes][2];  // [32-bit][mode][long reads]
  KernelFn rescan;                      // after them
  KernelFn front;                       // zero, plan, scan and scatter of a small batch
  KernelFn rerun[2];
  KernelFn zero, plan, scan, scatter;
  KernelTable();
};
const KernelTable& kernels();
hipError_t launch_pack2bit(const uint8_t* codes, int64_t n, uint32_t* words, hipStream_t s);
}  // namespace mica
