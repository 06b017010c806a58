// Host runtime of the DP-phase library: context, argument validation, device
// workspace, kernel plan table and the launch sequence behind the C ABI.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "ctx.h"
#include "dp_common.h"
#include "mica_dp.h"
#include "plan.h"

using namespace mica;

namespace mica {
thread_local std::string g_last_error;
mica_status_t fail(mica_status_t st, const std::string& msg) {
  g_last_error = msg;
  return st;
}
}  // namespace mica

namespace {
double bucket_cost(int b);
}

namespace mica {

void queue_order(uint32_t qorder[kNumBuckets], uint32_t persist_q[kQueueParts]) {
  int order[kNumBuckets];
  for (int b = 0; b < kNumBuckets; ++b) order[b] = b;
  // buckets of the persistent kernels first (per mode, long-read part
  // first), each part by descending item cost, then the plain buckets
  std::stable_sort(order, order + kNumBuckets, [](int x, int y) {
    if (queue_part(x) != queue_part(y)) return queue_part(x) < queue_part(y);
    return bucket_cost(x) > bucket_cost(y);
  });
  for (int q = 0; q < kQueueParts; ++q) persist_q[q] = 0;
  for (int b = 0; b < kNumBuckets; ++b)
    for (int q = queue_part(b); q + 1 < kQueueParts; ++q) persist_q[q + 1]++;
  for (int q = 0; q < kNumBuckets; ++q) qorder[q] = (uint32_t)order[q];
}

}  // namespace mica

namespace {

uint32_t* small_bcount(mica_ctx* c) { return c->d_small + small::kBcount; }
uint32_t* small_bstart(mica_ctx* c) { return c->d_small + small::kBstart; }
uint32_t* small_qstart(mica_ctx* c) { return c->d_small + small::kQstart; }
uint32_t* small_qorder(mica_ctx* c) { return c->d_small + small::kQorder; }
uint32_t* small_counters(mica_ctx* c) { return c->d_small + small::kCounters; }
uint32_t* small_bhead(mica_ctx* c) { return c->d_small + small::kBhead; }
uint32_t* small_scount(mica_ctx* c) { return c->d_small + small::kScount; }
uint32_t* small_sfill(mica_ctx* c) { return c->d_small + small::kSfill; }
uint32_t* small_fbcount(mica_ctx* c) { return c->d_small + small::kFbcount; }
uint32_t* small_sidehead(mica_ctx* c) { return c->d_small + small::kSidehead; }
constexpr size_t kSmallWords = small::kWords;

// cost of one work item of a bucket, for the descending work-queue order
double bucket_cost(int b) {
  const int kind = bucket_kind(b), cls = bucket_class(b), mode = bucket_mode(b);
  double c = class_rows(cls) * (class_lanes(cls) == 64 ? 1.5 : 1.0);
  if (mode == 1) c *= 1.25;
  if (kind == kK16Sat) c *= 1.1;
  if (kind == kK32) c *= 1.05;
  return c;
}

void default_plan(mica_ctx* c) {
  for (int m = 0; m <= kMaxM; ++m) c->class_of_m[m] = (uint8_t)default_class_of(m);
  c->class_dirty = true;
}

// same bounds as the device planner: can every cell stay inside int16?
// (extensions: start scores up to max_h0)
bool int16_always_safe(int max_m, int max_n, const mica_scoring_t& s, bool any_local, bool any_sg, bool any_ext,
                       int max_h0) {
  long hi = (long)s.match * (long)std::min(max_m, max_n);
  long lo = 0;
  if (any_sg) lo = std::min(lo, -(long)(2 * s.gap_open + (long)(max_m + 1) * s.gap_extend) - (kMaxM - 1));
  if (any_local) lo = std::min(lo, -(long)(s.gap_open + s.gap_extend) - (kMaxM - 1));
  if (any_ext) {
    hi = std::max(hi, (long)max_h0 + (long)s.match * (long)std::min(max_m, max_n));
    lo = std::min(lo, -3L * s.gap_open - (long)(max_m + max_n + 1) * s.gap_extend);
  }
  return hi <= 32767 - 8 && lo >= -32767 + 8;
}

mica_status_t ensure_pairs(mica_ctx* c, int64_t n) {
  if (n <= c->pair_cap) return MICA_OK;
  if (c->d_pairs) HIP_TRY(hipFree(c->d_pairs));
  c->d_pairs = nullptr;
  const int64_t cap = std::max<int64_t>(n, 1024);
  if (hipMalloc(&c->d_pairs, (size_t)cap * kPairLists * sizeof(uint32_t)) != hipSuccess) {
    c->pair_cap = 0;
    return fail(MICA_ERR_OUT_OF_MEMORY, "cannot allocate per-pair workspace");
  }
  c->pair_cap = cap;
  return MICA_OK;
}

mica_status_t ensure_scratch(mica_ctx* c, size_t bytes) {
  if (bytes <= c->scratch_cap) return MICA_OK;
  if (c->d_scratch) HIP_TRY(hipFree(c->d_scratch));
  c->d_scratch = nullptr;
  if (hipMalloc(&c->d_scratch, bytes) != hipSuccess) {
    c->scratch_cap = 0;
    return fail(MICA_ERR_OUT_OF_MEMORY, "cannot allocate traceback scratch");
  }
  c->scratch_cap = bytes;
  return MICA_OK;
}

hipError_t take_event(mica_ctx* c, hipEvent_t* e) {
  if (!c->ev_pool.empty()) {
    *e = c->ev_pool.back();
    c->ev_pool.pop_back();
    return hipSuccess;
  }
  return hipEventCreate(e);
}

hipError_t launch(KernelFn fn, unsigned blocks, unsigned threads, size_t shmem, hipStream_t s,
                  const Params* dp) {
  void* args[] = {(void*)&dp};
  return hipLaunchKernel((const void*)fn, dim3(blocks), dim3(threads), args, shmem, s);
}

hipKernelNodeParams node_params(const Launch& l, void** args) {
  hipKernelNodeParams p;
  std::memset(&p, 0, sizeof(p));
  p.func = (void*)l.fn;
  p.gridDim = dim3(l.grid);
  p.blockDim = dim3(l.block);
  p.sharedMemBytes = (unsigned)l.shmem;
  p.kernelParams = args;
  p.extra = nullptr;
  return p;
}

// Build the graph of a launch sequence: a chain of kernel nodes, with event
// record nodes around the fill launches when timing is on.
mica_status_t build_graph(mica_ctx* c, const std::vector<Launch>& seq, bool timing, const Params* dp,
                          hipEvent_t t0, hipEvent_t t1, mica_ctx::Graph* out) {
  mica_ctx::Graph g;
  HIP_TRY(hipGraphCreate(&g.graph, 0));
  hipGraphNode_t prev = nullptr;
  auto add_event = [&](hipEvent_t e, hipGraphNode_t* node) -> hipError_t {
    hipError_t err = hipGraphAddEventRecordNode(node, g.graph, prev ? &prev : nullptr, prev ? 1 : 0, e);
    if (err == hipSuccess) prev = *node;
    return err;
  };
  bool began = false;
  for (size_t i = 0; i < seq.size(); ++i) {
    if (timing && seq[i].fill && !began) {
      HIP_TRY(add_event(t0, &g.ev_begin));
      began = true;
    }
    void* args[] = {(void*)&dp};
    hipKernelNodeParams p = node_params(seq[i], args);
    hipGraphNode_t node;
    HIP_TRY(hipGraphAddKernelNode(&node, g.graph, prev ? &prev : nullptr, prev ? 1 : 0, &p));
    g.kernel_nodes.push_back(node);
    prev = node;
    const bool last_fill = seq[i].fill && (i + 1 == seq.size() || !seq[i + 1].fill);
    if (timing && last_fill) HIP_TRY(add_event(t1, &g.ev_end));
  }
  if (timing && !began) {  // no fill launch: the two events are adjacent
    HIP_TRY(add_event(t0, &g.ev_begin));
    HIP_TRY(add_event(t1, &g.ev_end));
  }
  HIP_TRY(hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0));
  c->graph_builds++;
  *out = g;
  return MICA_OK;
}

mica_status_t run_sequence(mica_ctx* c, const std::vector<Launch>& seq, const Params* dp, hipStream_t stream,
                           bool use_graph, hipEvent_t t0, hipEvent_t t1) {
  const bool timing = t0 != nullptr;
  if (!use_graph) {
    bool began = false;
    for (size_t i = 0; i < seq.size(); ++i) {
      if (timing && seq[i].fill && !began) {
        HIP_TRY(hipEventRecord(t0, stream));
        began = true;
      }
      HIP_TRY(launch(seq[i].fn, seq[i].grid, seq[i].block, seq[i].shmem, stream, dp));
      if (timing && seq[i].fill && (i + 1 == seq.size() || !seq[i + 1].fill)) HIP_TRY(hipEventRecord(t1, stream));
    }
    if (timing && !began) {
      HIP_TRY(hipEventRecord(t0, stream));
      HIP_TRY(hipEventRecord(t1, stream));
    }
    return MICA_OK;
  }
  // (grid, block and LDS are set on the graph: the LDS of the seeded kernels
  // follows the batch's length bounds)
  std::vector<uint64_t> key;
  key.push_back(timing ? 1 : 0);
  for (const Launch& l : seq) key.push_back((uint64_t)(uintptr_t)l.fn << 1 | (l.fill ? 1 : 0));
  auto it = c->graphs.find(key);
  if (it == c->graphs.end()) {
    if (c->graphs.size() >= kMaxGraphs) {
      auto old = c->graphs.begin();
      for (auto g = c->graphs.begin(); g != c->graphs.end(); ++g)
        if (g->second.used < old->second.used) old = g;
      HIP_TRY(hipDeviceSynchronize());  // it may still run
      (void)hipGraphExecDestroy(old->second.exec);
      (void)hipGraphDestroy(old->second.graph);
      c->graphs.erase(old);
    }
    mica_ctx::Graph g;
    mica_status_t st = build_graph(c, seq, timing, dp, t0, t1, &g);
    if (st != MICA_OK) return st;
    it = c->graphs.emplace(std::move(key), g).first;
  } else {
    mica_ctx::Graph& g = it->second;
    for (size_t i = 0; i < seq.size(); ++i) {
      void* args[] = {(void*)&dp};
      hipKernelNodeParams p = node_params(seq[i], args);
      HIP_TRY(hipGraphExecKernelNodeSetParams(g.exec, g.kernel_nodes[i], &p));
    }
    if (timing) {
      HIP_TRY(hipGraphExecEventRecordNodeSetEvent(g.exec, g.ev_begin, t0));
      HIP_TRY(hipGraphExecEventRecordNodeSetEvent(g.exec, g.ev_end, t1));
    }
  }
  it->second.used = ++c->graph_launches;
  HIP_TRY(hipGraphLaunch(it->second.exec, stream));
  return MICA_OK;
}

}  // namespace

namespace mica {

mica_status_t check_batch(const mica_batch_t* b, const mica_scoring_t* s, uint32_t flags, uint32_t known) {
  if (!b || !s) return fail(MICA_ERR_INVALID_ARG, "NULL batch or scoring");
  if (flags & ~known) return fail(MICA_ERR_INVALID_ARG, "unknown flag bits");
  if (s->match < 1 || s->match > 4096 || s->mismatch > 0 || s->mismatch < -4096 || s->gap_open < 0 ||
      s->gap_open > 4096 || s->gap_extend < 1 || s->gap_extend > 4096)
    return fail(MICA_ERR_INVALID_ARG, "scoring outside its limits");
  if (b->n_pairs < 0) return fail(MICA_ERR_INVALID_ARG, "n_pairs < 0");
  if (b->n_pairs > 0xFFFFFFF0ll) return fail(MICA_ERR_LIMIT, "too many pairs in one batch");
  if (b->default_mode < 0 || b->default_mode > 2) return fail(MICA_ERR_INVALID_ARG, "bad default_mode");
  if (b->mode_mask < 0 || b->mode_mask > 7) return fail(MICA_ERR_INVALID_ARG, "bad mode_mask");
  if (b->ext_clip < 0 || b->ext_clip > kMaxH0 || b->ext_default_h0 < 0 || b->ext_default_h0 > kMaxH0)
    return fail(MICA_ERR_INVALID_ARG, "extension start score or clipping penalty outside 0..2^20");
  if (b->max_read_len < 0 || b->max_read_len > kMaxM || b->max_win_len < 0 || b->max_win_len > kMaxN)
    return fail(MICA_ERR_LIMIT, "max_read_len / max_win_len beyond the library limits");
  if (b->min_read_len < 0 || b->min_read_len > b->max_read_len)
    return fail(MICA_ERR_INVALID_ARG, "min_read_len outside [0, max_read_len]");
  if (b->max_ext_h0 < 0 || b->max_ext_h0 > kMaxH0)
    return fail(MICA_ERR_INVALID_ARG, "max_ext_h0 outside 0..2^20");
  const bool want_cigar = flags & MICA_OUT_CIGAR;
  const bool want_start = want_cigar || (flags & MICA_OUT_START);
  if (b->n_pairs == 0) return MICA_OK;
  if (!b->ref2b || !b->win_off || !b->win_len || !b->reads2b || !b->read_off || !b->read_len ||
      !b->score || !b->read_end || !b->ref_end || !b->status)
    return fail(MICA_ERR_INVALID_ARG, "NULL input or output pointer");
  if (want_start && (!b->read_start || !b->ref_start))
    return fail(MICA_ERR_INVALID_ARG, "read_start / ref_start required for start or CIGAR output");
  if (want_cigar && (!b->n_cigar || b->cigar_cap < 0 || (b->cigar_cap > 0 && !b->cigar)))
    return fail(MICA_ERR_INVALID_ARG, "cigar / n_cigar / cigar_cap invalid");
  return MICA_OK;
}

namespace {
struct OccEntry {
  int device;
  KernelFn fn;
  int threads;
  size_t shmem;
  int blocks;
};
constexpr int kOccCache = 1024;
OccEntry g_occ[kOccCache];
int g_n_occ = 0;
std::mutex g_occ_mu;
}  // namespace

mica_status_t kernel_occupancy(int device, KernelFn fn, int threads, size_t shmem, int* blocks) {
  std::lock_guard<std::mutex> g(g_occ_mu);
  for (int i = 0; i < g_n_occ; ++i)
    if (g_occ[i].device == device && g_occ[i].fn == fn && g_occ[i].threads == threads && g_occ[i].shmem == shmem) {
      *blocks = g_occ[i].blocks;
      return MICA_OK;
    }
  int nb = 0;
  HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)fn, threads, shmem));
  nb = std::max(nb, 1);
  if (g_n_occ < kOccCache) g_occ[g_n_occ++] = {device, fn, threads, shmem, nb};
  *blocks = nb;
  return MICA_OK;
}

namespace {

// The band kernels of a batch.  Plain launches compute every table in full
// (they are what the band kernels are compared with), and reads too short
// for a certificate only pay for the scan.
mica_status_t plan_prune(int device, const uint8_t* class_of_m, const mica_batch_t* b, const mica_scoring_t& s, uint32_t flags, int traced,
                         const bool any_mode[kNumModes], FillPlan* fp) {
  fp->n_prune = 0;
  if (flags & MICA_PLAIN_LAUNCH) return MICA_OK;
  // Scores alone take one pass of the fill: where that does not fill the GPU
  // several times over, one item's latency is the time of both ways (1,000
  // pairs of 150 x 200 in 32 bits: 60 us in the fill, 170 us here), and a scan
  // that finds the reads too noisy costs some 50 us (70,000 of 60 x 120, 6%
  // errors: 261 us without it, 304 with it; 140,000 of 150 x 300: 1.20, 1.26 ms).
  if (!traced && (b->n_pairs < 65536 || (double)b->n_pairs * b->max_read_len * b->max_win_len < 3e9)) return MICA_OK;
  // four parts at least: 20,000 traced pairs of 30 x 109 take 157 us here and 176
  // in the fills without errors, 262 and 185 with 5%
  const int parts = b->max_read_len / kSeed;
  if (!any_mode[MICA_MODE_EXTEND] && parts < 4) return MICA_OK;
  // Traced reads of few parts are often left, and a fill of some thousands of them
  // is as quick as one of those left (60 x 154 local, 20,000: 257 us without
  // errors, 278 with 5%; here 197 and 385; 40,000: 346 and 378; here 228 and 424).
  if (traced && !any_mode[MICA_MODE_EXTEND] && b->max_read_len < kFewPartsRead && b->n_pairs >= 4096 &&
      b->n_pairs < 32768)
    return MICA_OK;
  // (the pairs left run in up to 256 dummy rows, more than the planner's 16-bit
  // check of short reads allows for)
  if (!(flags & MICA_FORCE_INT32) && 2L * s.gap_open + (long)(kMaxM + 1) * s.gap_extend + 256 > 32767 - 8) return MICA_OK;
  Params& S = fp->prune_shape;
  std::memset(&S, 0, sizeof(S));
  const int m = b->max_read_len, n = b->max_win_len;
  S.pr_costs = seed_costs(s.match, s.mismatch, s.gap_open, s.gap_extend, kMaxM / kSeed);
  S.pr_win_words = (n + 15) / 16 + 2;
  S.pr_read_words = (m + 15) / 16 + 1;
  S.pr_part_words = std::max(4, (m / kSeed + 3) / 4 * 4);
  S.pr_rows = (m + 1) / 2 * 2;
  S.pr_group_words = S.pr_rows + (m + kBandMaxW + 2) / 2;
  S.pr_scan_words = kScanStaticWords + 8 * (S.pr_win_words + S.pr_read_words + S.pr_part_words);
  // (sequences of the two pairs of a group: read and band, from any base)
  S.pr_raw_off = kBandStaticWords + (int)align_up((size_t)4 * S.pr_group_words, 4);
  S.pr_raw_words = 2 * ((m + 15) / 16 + (m + kBandMaxW + 15) / 16);
  S.pr_band_words = S.pr_raw_off + (int)align_up((size_t)4 * S.pr_raw_words, 4);
  // direction bits of 64 lanes, two rows a word; CIGAR staging of 8 pairs
  S.pr_rec_bytes = traced ? (uint64_t)(m / 2 + 1) * 256 : 0;
  S.pr_slot_bytes = std::max<uint64_t>(
      align_up(S.pr_rec_bytes + (traced ? (size_t)8 * (size_t)(m + n + 2) * 4 : 0), 256), 256);
  // blocks of four waves, or fewer where their LDS would pass 62 KB
  auto block = [](int words, int* threads, size_t* shmem) {
    const size_t bytes = (size_t)words * 4;
    *threads = bytes * 4 <= (size_t)63488 ? 256 : (bytes * 2 <= (size_t)63488 ? 128 : 64);
    *shmem = align_up(bytes * (size_t)(*threads / 64), 2048);
  };
  block(S.pr_scan_words, &fp->scan_threads, &fp->scan_shmem);
  block(S.pr_band_words, &fp->prune_threads, &fp->prune_shmem);
  const int wide = (flags & MICA_FORCE_INT32) ? 1 : 0;
  fp->scan_fn = kernels().seed_scan[traced][wide];
  fp->sample_fn = kernels().seed_sample[traced][wide];
  // (an extension needs no part, so its band is nearly always known)
  fp->sampled = b->n_pairs >= kSamplePairs && (!traced || m < kSampleRead) &&
                (any_mode[MICA_MODE_SEMIGLOBAL] || any_mode[MICA_MODE_LOCAL]);
  int n_prune = 0;
  for (int md = 0; md < kNumModes; ++md) {
    if (!any_mode[md]) continue;
    fp->prune[n_prune] = kernels().seed_band[traced][wide][md];
    mica_status_t st =
        kernel_occupancy(device, fp->prune[n_prune], fp->prune_threads, fp->prune_shmem, &fp->prune_occ[n_prune]);
    if (st != MICA_OK) return st;
    ++n_prune;
  }
  fp->n_prune = n_prune;
  S.left_full_ = traced && m > kLeftFullRead ? 1 : 0;
  fp->n_left = 0;
  fp->left_pairs = wide ? 1 : 2;
  // (their items have 128 rows at least, whatever the reads: 9,000 items of 60
  // bases take 250 us there, 221 in a fill and its side lists)
  fp->left_rounds = m <= 64 && (any_mode[MICA_MODE_SEMIGLOBAL] || any_mode[MICA_MODE_LOCAL]) ? 2 : 4;
  bool short_class[kNumClasses] = {};
  for (int r = std::max(1, b->min_read_len); r <= m; ++r) short_class[class_of_m[r]] = !left_long(class_of_m[r]);
  fp->left_buckets = 0;
  for (int c = 0; c < kNumClasses; ++c) {
    for (int md = 0; md < kNumModes; ++md) fp->left_buckets += short_class[c] && any_mode[md] ? 1 : 0;
  }
  for (int md = 0; md < kNumModes && traced; ++md)
    for (int lng = 0; lng < 2; ++lng) {
      bool used = false;
      for (int r = std::max(1, b->min_read_len); r <= m; ++r) used |= (left_long(class_of_m[r]) ? 1 : 0) == lng;
      if (!any_mode[md] || !used) continue;
      const int i = fp->n_left++;
      fp->left[i] = kernels().seed_left[wide][md][lng];
      fp->left_long_reads[i] = lng;
      mica_status_t st = kernel_occupancy(device, fp->left[i], 256, kFillShmem, &fp->left_occ[i]);
      if (st != MICA_OK) return st;
    }
  return MICA_OK;
}

}  // namespace

int64_t prune_slots(const FillPlan& fp, int n_cu, int64_t n_pairs, size_t bytes) {
  if (fp.n_prune == 0) return 0;
  const int64_t per_block = fp.prune_threads / 64;
  int occ = 1;
  for (int i = 0; i < fp.n_prune; ++i) occ = std::max(occ, fp.prune_occ[i]);
  int64_t slots = (int64_t)occ * n_cu * per_block;
  // the bands of a mode: at most one partial item per class and list
  slots = std::min(slots, (int64_t)align_up((size_t)(n_pairs / 4 + 2 * kNumClasses), (size_t)per_block));
  // (a slot and a block here are no larger than the fills', so the memory of a
  // block of fills, which every call has, holds a block of these)
  return std::min(slots, (int64_t)(bytes / fp.prune_shape.pr_slot_bytes) / per_block * per_block);
}

// Items a wave of the scan takes: about two waves per SIMD, and at most one list
// request per kScanChunk items.
static int scan_chunk(int n_cu, int64_t n_pairs) {
  const int64_t per_wave = n_pairs / kPruneItem / ((int64_t)n_cu * 8);
  return (int)std::max<int64_t>(1, std::min<int64_t>(kScanChunk, per_wave));
}

// the waves of a k_seed_left launch: an item each, as far as they are resident
static int64_t left_waves(const FillPlan& fp, int i, int n_cu, int64_t n_pairs, int64_t fill_slots) {
  const int64_t items = n_pairs / fp.left_pairs + kNumClasses;  // a partial one per class
  const int64_t want = std::min<int64_t>((int64_t)align_up((size_t)items, kWavesPerBlock),
                                         (int64_t)fp.left_occ[i] * n_cu * kWavesPerBlock);
  return std::min(want, fill_slots / kWavesPerBlock * kWavesPerBlock);
}
// and of the short-read ones together
static int64_t left_short_waves(const FillPlan& fp, int n_cu, int64_t n_pairs, int64_t fill_slots) {
  int64_t waves = 0;
  for (int i = 0; i < fp.n_left; ++i)
    if (!fp.left_long_reads[i]) waves = std::max(waves, left_waves(fp, i, n_cu, n_pairs, fill_slots));
  return waves;
}

void prune_params(Params* P, const FillPlan& fp, int n_cu, int64_t slots, int64_t fill_slots, uint32_t* rerun,
                  uint32_t* wlist, uint32_t* small) {
  P->lcount = small + small::kLcount;
  P->left_limit = (int32_t)(fp.left_rounds * left_short_waves(fp, n_cu, P->n_pairs, fill_slots));
  P->pr_sampled = fp.sampled ? 1 : 0;
  P->pr_sample_waves = fp.scan_threads / 64;
  P->pr_chunk = scan_chunk(n_cu, P->n_pairs);
  const Params& S = fp.prune_shape;
  P->presorted = rerun;
  P->rcount = small + small::kRcount;
  P->nbcount = small + small::kNbcount;
  P->w32count = small + small::kW32count;
  P->w64count = small + small::kW64count;
  P->wlist = wlist;
  P->pqstart = small + small::kPqstart;
  P->left_full_ = S.left_full_;
  P->pr_slot_bytes = S.pr_slot_bytes;
  P->pr_rec_bytes = S.pr_rec_bytes;
  P->pr_slots = (int32_t)slots;
  P->pr_scan_words = S.pr_scan_words;
  P->pr_band_words = S.pr_band_words;
  P->pr_win_words = S.pr_win_words;
  P->pr_read_words = S.pr_read_words;
  P->pr_part_words = S.pr_part_words;
  P->pr_rows = S.pr_rows;
  P->pr_group_words = S.pr_group_words;
  P->pr_raw_off = S.pr_raw_off;
  P->pr_raw_words = S.pr_raw_words;
  P->pr_costs = S.pr_costs;
}

void launch_sequence(const FillPlan& fp, int n_cu, int64_t n_pairs, int64_t slots, int64_t pr_slots,
                     std::vector<Launch>* seq) {
  const KernelTable& K = kernels();
  if (n_pairs <= kFrontPairs) {
    seq->push_back({K.front, 1, 256, 0, false});
  } else {
    const unsigned blocks = (unsigned)((n_pairs + kPlanPairsPerBlock - 1) / kPlanPairsPerBlock);
    seq->push_back({K.zero, 1, 256, 0, false});
    seq->push_back({K.plan, blocks, kPlanThreads, 0, false});
    if (pr_slots > 0 && fp.sampled)
      seq->push_back({fp.sample_fn, 1 + (unsigned)(kSampleWaves * 64 / fp.scan_threads), kScanThreads, fp.scan_shmem, false});
    else
      seq->push_back({K.scan, 1, kScanThreads, 0, false});
    seq->push_back({K.scatter, blocks, kPlanThreads, 0, false});
  }
  if (pr_slots > 0) {
    // an item per wave, at most one partial item per class and mode
    const int64_t items = n_pairs / kPruneItem + kNumModes * kNumClasses;
    const int64_t per_block = fp.prune_threads / 64;
    const int64_t per_scan = fp.scan_threads / 64 * scan_chunk(n_cu, n_pairs);
    const int64_t blocks = (std::min(items, n_pairs) + per_scan - 1) / per_scan;
    seq->push_back({fp.scan_fn, (unsigned)blocks, (unsigned)fp.scan_threads, fp.scan_shmem, true});
    for (int i = 0; i < fp.n_prune; ++i) {
      const int64_t bands = std::min<int64_t>((int64_t)fp.prune_occ[i] * n_cu, pr_slots / per_block);
      seq->push_back({fp.prune[i], (unsigned)bands, (unsigned)fp.prune_threads, fp.prune_shmem, true});
    }
    seq->push_back({K.rescan, 1, 256, 0, true});
  }
  bool lw_all = false;
  if (pr_slots > 0) {
    // (can the short reads' launches take whatever is left?)
    const uint64_t lw = (uint64_t)left_short_waves(fp, n_cu, n_pairs, slots);
    const uint64_t per = (uint64_t)fp.left_pairs, n = (uint64_t)n_pairs;
    const uint64_t most = std::min(n, (n + (per - 1) * (uint64_t)fp.left_buckets) / per);
    lw_all = most <= fp.left_rounds * lw;
    for (int i = 0; i < fp.n_left; ++i) {
      const int64_t waves = left_waves(fp, i, n_cu, n_pairs, slots);
      seq->push_back({fp.left[i], (unsigned)(waves / kWavesPerBlock), 256, kFillShmem, true});
    }
  }
  for (int i = 0; i < fp.n; ++i) {
    if (lw_all && fp.spare[i]) continue;
    // each fill kernel gets the blocks it keeps resident (its waves index
    // the first slots of the scratch)
    const int64_t blocks = std::min<int64_t>((int64_t)fp.occ[i] * n_cu, slots / kWavesPerBlock);
    if (fp.single[i]) seq->push_back({fp.fn[i], 1, 256, 0, true});
    else seq->push_back({fp.fn[i], (unsigned)std::max<int64_t>(blocks, 1), 256, kFillShmem, true});
  }
}

mica_status_t plan_fills(int device, const uint8_t* class_of_m, const mica_batch_t* b, const mica_scoring_t* s,
                         uint32_t flags, FillPlan* out) {
  const KernelTable& K = kernels();
  FillPlan& fp = *out;
  fp.n = 0;
  for (int i = 0; i < kMaxFills; ++i) fp.single[i] = fp.spare[i] = false;
  fp.occ_max = 1;
  const int max_m = b->max_read_len, max_n = b->max_win_len;
  const int d = (flags & (MICA_OUT_CIGAR | MICA_OUT_START)) ? 1 : 0;
  const bool forced = flags & MICA_FORCE_INT32;
  const int mode_mask = b->mode ? (b->mode_mask ? b->mode_mask : 7) : 1 << b->default_mode;
  fp.mode_mask = mode_mask;
  const bool any_sg = mode_mask & 1, any_local = mode_mask & 2, any_ext = mode_mask & 4;
  const bool any_mode[3] = {any_sg, any_local, any_ext};
  // extensions start from per-pair scores the host does not read: without
  // a bound on them their saturating variants are always available
  const bool may_sat = !forced && ((any_ext && b->max_ext_h0 == 0) ||
                                   !int16_always_safe(max_m, max_n, *s, any_local, any_sg, any_ext, b->max_ext_h0));
  const bool plain = flags & MICA_PLAIN_LAUNCH;
  mica_status_t ps = plan_prune(device, class_of_m, b, *s, flags, d, any_mode, &fp);
  if (ps != MICA_OK) return ps;
  // what the band kernels leave of their kinds with a traceback: reads of the
  // long classes to k_seed_left, others there (spare) or, where they are many,
  // to the side lists or the fills
  auto seeded = [&](int kind) { return fp.n_prune > 0 && d && prune_kind(kind); };
  auto filled = [&](int kind, int md) { return !seeded(kind) || !left_full(&fp.prune_shape, md); };
  bool cls_used[kNumClasses] = {};
  for (int m = std::max(1, b->min_read_len); m <= max_m; ++m) cls_used[class_of_m[m]] = true;
  // a batch of one persistent class gains nothing from the persistent
  // kernels (they balance classes against each other) and its plain kernel
  // is compiled for that class alone
  int n_persist_cls = 0;
  for (int cls = 0; cls <= kPersistMaxClass; ++cls)
    if (cls_used[cls] && class_lanes(cls) == 16) ++n_persist_cls;
  const bool persist = !plain && !forced && n_persist_cls > 1;
  bool part_used[2] = {false, false};
  for (int cls = 0; cls <= kPersistMaxClass; ++cls)
    if (cls_used[cls] && class_lanes(cls) == 16) part_used[persist_part(cls)] = true;
  if (persist) {
    // persistent parts in queue order: per mode, long reads first
    for (int md = 0; md < kNumModes; ++md) {
      if (!any_mode[md]) continue;
      if (!filled(kK16, md)) continue;
      for (int part : {1, 0}) {
        if (!part_used[part]) continue;
        fp.spare[fp.n] = seeded(kK16);
        fp.fn[fp.n++] = K.persistent[d][md][part];
      }
    }
  }
  const bool any_persistent = fp.n > 0;
  // plain launches: every bucket in plain mode, else the buckets the
  // persistent kernels do not serve
  auto plain_buckets = [&](const KernelFn* table, bool side) {
    for (int kind = 0; kind < kNumKinds; ++kind) {
      if (forced != (kind == kK32)) continue;
      if (kind == kK16Sat && !may_sat) continue;
      for (int cls = 0; cls < kNumClasses; ++cls) {
        if (!cls_used[cls]) continue;
        for (int md = 0; md < kNumModes; ++md) {
          if (!any_mode[md]) continue;
          const int bk = bucket_id(kind, cls, md);
          if (persist && persistent_bucket(bk)) continue;
          if (seeded(kind) && left_long(cls)) continue;
          if (!side && !filled(kind, md)) continue;
          fp.spare[fp.n] = seeded(kind);
          fp.fn[fp.n++] = table[bk];
        }
      }
    }
  };
  plain_buckets(K.bucket[d], false);
  // the side lists of the banded fills (pairs whose band was too wide: the
  // full traceback; bands of 17-64 diagonals: the band refill), after every
  // banded fill: persistent kernels over the persistent buckets (one queue
  // per mode and class part) and one launch per other bucket
  if (d) {
    if (persist) {
      // (without a fill of these buckets the scan after the band kernels has
      // done it)
      if (any_persistent) {
        fp.single[fp.n] = true;
        fp.spare[fp.n] = seeded(kK16);
        fp.fn[fp.n++] = K.sidescan;
      }
      for (int md = 0; md < kNumModes; ++md) {
        if (!any_mode[md]) continue;
        for (int part : {1, 0}) {
          if (!part_used[part]) continue;
          fp.spare[fp.n] = seeded(kK16);
          fp.fn[fp.n++] = K.side_persistent[md][part];
        }
      }
    }
    plain_buckets(K.side, true);
  }
  if (may_sat) fp.fn[fp.n++] = K.rerun[d];
  for (int i = 0; i < fp.n; ++i) {
    if (fp.single[i]) {
      fp.occ[i] = 1;
      continue;
    }
    mica_status_t st = kernel_occupancy(device, fp.fn[i], 256, kFillShmem, &fp.occ[i]);
    if (st != MICA_OK) return st;
    fp.occ_max = std::max(fp.occ_max, fp.occ[i]);
  }
  for (int i = 0; fp.n_prune && i < fp.n_left; ++i) fp.occ_max = std::max(fp.occ_max, fp.left_occ[i]);
  return MICA_OK;
}

SlotShape slot_shape(const mica_batch_t* b, uint32_t flags) {
  SlotShape sh;
  const int d = (flags & (MICA_OUT_CIGAR | MICA_OUT_START)) ? 1 : 0;
  // the full traceback's direction words (steps x 64 lanes x 16 B), or the
  // band records (two rows per word, 4 strips x 64 lanes), whichever is larger
  sh.dir_bytes = d ? std::max((size_t)(b->max_win_len + 64) * 64 * 16, (size_t)(b->max_read_len / 2 + 1) * 1024) : 0;
  sh.stage_stride = b->max_read_len + b->max_win_len + 2;
  // then a wave's pending pairs (kPendWords words)
  const size_t stage_bytes = d ? (size_t)8 * sh.stage_stride * 4 + kPendWords * 4 : 0;
  sh.slot_bytes = std::max<size_t>(align_up(sh.dir_bytes + stage_bytes, 256), 256);
  return sh;
}

void batch_params(Params* P_, const mica_batch_t* b, const mica_scoring_t* s, uint32_t flags, int mode_mask) {
  Params& P = *P_;
  const bool want_cigar = flags & MICA_OUT_CIGAR;
  const bool want_start = want_cigar || (flags & MICA_OUT_START);
  std::memset(&P, 0, sizeof(P));
  P.ref2b = b->ref2b;
  P.ref_len = b->ref_len;
  P.win_off = b->win_off;
  P.win_len = b->win_len;
  P.reads2b = b->reads2b;
  P.reads_len = b->reads_len;
  P.read_off = b->read_off;
  P.read_len = b->read_len;
  P.mode = b->mode;
  P.default_mode = b->default_mode;
  P.ext_h0 = b->ext_h0;
  P.ext_default_h0 = b->ext_default_h0;
  P.max_h0 = b->max_ext_h0 ? b->max_ext_h0 : kMaxH0;
  P.ext_clip = b->ext_clip;
  P.mode_mask = mode_mask;
  P.max_m = b->max_read_len;
  P.min_m = b->min_read_len;
  P.max_n = b->max_win_len;
  P.n_pairs = b->n_pairs;
  P.score = b->score;
  P.read_end = b->read_end;
  P.ref_end = b->ref_end;
  P.read_start = want_start ? b->read_start : nullptr;
  P.ref_start = want_start ? b->ref_start : nullptr;
  P.cigar = want_cigar ? b->cigar : nullptr;
  P.cigar_cap = want_cigar ? b->cigar_cap : 0;
  P.n_cigar = want_cigar ? b->n_cigar : nullptr;
  P.status = b->status;
  P.sa = s->match;
  P.sb = s->mismatch;
  P.so = s->gap_open;
  P.se = s->gap_extend;
  P.flags = (want_start ? kOutStart : 0u) | (want_cigar ? kOutCigar : 0u) |
            ((flags & MICA_FORCE_INT32) ? kForceInt32 : 0u);
}

}  // namespace mica

extern "C" {

const char* mica_last_error(void) { return g_last_error.c_str(); }

mica_status_t mica_ctx_create(int hip_device, size_t workspace_bytes, mica_ctx_t* out) {
  if (!out) return fail(MICA_ERR_INVALID_ARG, "out is NULL");
  *out = nullptr;
  int ndev = 0;
  HIP_TRY(hipGetDeviceCount(&ndev));
  if (hip_device < 0 || hip_device >= ndev) return fail(MICA_ERR_INVALID_ARG, "no such HIP device");
  HIP_TRY(hipSetDevice(hip_device));
  mica_ctx* c = new mica_ctx();
  c->device = hip_device;
  if (workspace_bytes) c->ws_cap = workspace_bytes;
  hipDeviceProp_t prop;
  HIP_TRY(hipGetDeviceProperties(&prop, hip_device));
  c->n_cu = prop.multiProcessorCount;
  c->arch = prop.gcnArchName;
  {
    const size_t colon = c->arch.find(':');
    if (colon != std::string::npos) c->arch.resize(colon);
  }
  HIP_TRY(hipMalloc(&c->d_params, sizeof(Params) * kParamRing));
  HIP_TRY(hipMalloc(&c->d_small, kSmallWords * sizeof(uint32_t)));
  HIP_TRY(hipMalloc(&c->d_class, kMaxM + 1));
  HIP_TRY(hipHostMalloc((void**)&c->h_params, sizeof(Params) * kParamRing, hipHostMallocDefault));
  for (int i = 0; i < kParamRing; ++i) HIP_TRY(hipEventCreateWithFlags(&c->ev[i], hipEventDisableTiming));
  default_plan(c);
  queue_order(c->qorder, c->persist_q);
  HIP_TRY(hipMemcpy(small_qorder(c), c->qorder, sizeof(c->qorder), hipMemcpyHostToDevice));
  HIP_TRY(hipMemcpy(c->d_class, c->class_of_m, kMaxM + 1, hipMemcpyHostToDevice));
  c->class_dirty = false;
  *out = c;
  return MICA_OK;
}

mica_status_t mica_ctx_destroy(mica_ctx_t c) {
  if (!c) return MICA_OK;
  (void)hipSetDevice(c->device);
  (void)hipDeviceSynchronize();
  for (int i = 0; i < kParamRing; ++i)
    if (c->ev[i]) (void)hipEventDestroy(c->ev[i]);
  if (c->h_params) (void)hipHostFree(c->h_params);
  if (c->d_params) (void)hipFree(c->d_params);
  if (c->d_small) (void)hipFree(c->d_small);
  if (c->d_class) (void)hipFree(c->d_class);
  if (c->d_pairs) (void)hipFree(c->d_pairs);
  if (c->d_scratch) (void)hipFree(c->d_scratch);
  for (auto& pr : c->ev_pending) {
    (void)hipEventDestroy(pr.first);
    (void)hipEventDestroy(pr.second);
  }
  for (auto e : c->ev_pool) (void)hipEventDestroy(e);
  for (auto& kv : c->graphs) {
    if (kv.second.exec) (void)hipGraphExecDestroy(kv.second.exec);
    if (kv.second.graph) (void)hipGraphDestroy(kv.second.graph);
  }
  delete c;
  return MICA_OK;
}

mica_status_t mica_ctx_set_plan(mica_ctx_t c, int32_t m_lo, int32_t m_hi, int32_t lanes, int32_t rows) {
  if (!c) return fail(MICA_ERR_INVALID_ARG, "ctx is NULL");
  if (m_lo < 1 || m_hi > kMaxM || m_lo > m_hi) return fail(MICA_ERR_INVALID_ARG, "bad read-length range");
  const int cls = class_of(lanes, rows);
  if (cls < 0) return fail(MICA_ERR_INVALID_ARG, "unsupported (lanes, rows)");
  if (lanes * rows < m_hi) return fail(MICA_ERR_INVALID_ARG, "lanes * rows must cover m_hi");
  HIP_TRY(hipSetDevice(c->device));
  // a batch still queued on any stream reads the device table when its
  // planning kernel runs, but its fill kernels were chosen from the host
  // table when it was enqueued: let every such batch finish first
  HIP_TRY(hipDeviceSynchronize());
  for (int m = m_lo; m <= m_hi; ++m) c->class_of_m[m] = (uint8_t)cls;
  HIP_TRY(hipMemcpy(c->d_class, c->class_of_m, kMaxM + 1, hipMemcpyHostToDevice));
  return MICA_OK;
}

mica_status_t mica_pack_2bit(const uint8_t* codes, int64_t n_bases, uint32_t* words, void* stream) {
  if (n_bases < 0) return fail(MICA_ERR_INVALID_ARG, "n_bases < 0");
  if (n_bases > 0 && (!codes || !words)) return fail(MICA_ERR_INVALID_ARG, "NULL pointer");
  HIP_TRY(launch_pack2bit(codes, n_bases, words, (hipStream_t)stream));
  return MICA_OK;
}

mica_status_t mica_dp_align_batch(mica_ctx_t c, const mica_batch_t* b, const mica_scoring_t* s,
                                  uint32_t flags, void* stream_) {
  if (!c) return fail(MICA_ERR_INVALID_ARG, "NULL ctx");
  const uint32_t known = MICA_OUT_START | MICA_OUT_CIGAR | MICA_FORCE_INT32 | MICA_PLAIN_LAUNCH | MICA_NO_GRAPH;
  mica_status_t st = check_batch(b, s, flags, known);
  if (st != MICA_OK) return st;
  if (b->n_pairs == 0) return MICA_OK;
  hipStream_t stream = (hipStream_t)stream_;
  HIP_TRY(hipSetDevice(c->device));

  st = ensure_pairs(c, b->n_pairs);
  if (st != MICA_OK) return st;

  // fill launches of this batch
  FillPlan fp;
  st = plan_fills(c->device, c->class_of_m, b, s, flags, &fp);
  if (st != MICA_OK) return st;

  // scratch: direction bits of a resident wave (steps x 64 lanes x 16 B) +
  // CIGAR staging, for as many waves as the most occupant fill kernel keeps
  // resident
  const SlotShape sh = slot_shape(b, flags);
  int64_t slots = (int64_t)fp.occ_max * c->n_cu * kWavesPerBlock;
  const int64_t by_ws = (int64_t)(c->ws_cap / sh.slot_bytes);
  slots = std::min(slots, by_ws);
  const int64_t need = (b->n_pairs + 1) / 2 + 3;  // upper bound of work items
  slots = std::min(slots, need);
  slots = std::max<int64_t>(align_up((size_t)std::max<int64_t>(slots, 1), kWavesPerBlock), kWavesPerBlock);
  if ((size_t)slots * sh.slot_bytes > c->ws_cap && slots > kWavesPerBlock)
    slots = (int64_t)(c->ws_cap / sh.slot_bytes) / kWavesPerBlock * kWavesPerBlock;
  if (slots < kWavesPerBlock) return fail(MICA_ERR_OUT_OF_MEMORY, "workspace too small for one block");
  // the band kernels run before the fills, in the same memory: under the cap, or
  // in the one block of fills that a smaller cap still gets
  const int64_t pr_want =
      prune_slots(fp, c->n_cu, b->n_pairs, std::max(c->ws_cap, (size_t)slots * sh.slot_bytes));
  // (the fills that the band kernels replace are not among the launches)
  if (fp.n_prune > 0 && pr_want == 0) return fail(MICA_ERR_OUT_OF_MEMORY, "workspace too small for the band kernels");
  const size_t scratch_bytes =
      std::max((size_t)slots * sh.slot_bytes, (size_t)pr_want * (size_t)fp.prune_shape.pr_slot_bytes);
  st = ensure_scratch(c, scratch_bytes);
  if (st != MICA_OK) return st;

  // parameter block (pinned ring slot, copied on the stream)
  const int rp = c->ring_pos;
  c->ring_pos = (c->ring_pos + 1) % kParamRing;
  if (c->ev_used[rp]) HIP_TRY(hipEventSynchronize(c->ev[rp]));
  Params& P = c->h_params[rp];
  batch_params(&P, b, s, flags, fp.mode_mask);
  P.bucket_of = c->d_pairs;
  P.sorted = c->d_pairs + c->pair_cap;
  P.rerun = c->d_pairs + 2 * c->pair_cap;
  P.fbsorted = c->d_pairs + 3 * c->pair_cap;
  P.fbcount = small_fbcount(c);
  P.sidehead = small_sidehead(c);
  P.fbqstart = c->d_small + small::kFbqstart;
  P.dbsorted = c->d_pairs + 4 * c->pair_cap;
  P.dbcount = c->d_small + small::kDbcount;
  P.dbwide = c->d_small + small::kDbwide;
  P.dbqstart = c->d_small + small::kDbqstart;
  P.bcount = small_bcount(c);
  P.bstart = small_bstart(c);
  P.scount = small_scount(c);
  P.sfill = small_sfill(c);
  P.qstart = small_qstart(c);
  P.qorder = small_qorder(c);
  P.class_of_m = c->d_class;
  P.counters = small_counters(c);
  P.bhead = small_bhead(c);
  P.scratch = c->d_scratch;
  P.slot_bytes = sh.slot_bytes;
  P.dir_bytes = sh.dir_bytes;
  P.stage_stride = sh.stage_stride;
  P.n_slots = (int32_t)slots;
  for (int i = 0; i < kQueueParts; ++i) P.persist_q[i] = c->persist_q[i];
  if (pr_want > 0) prune_params(&P, fp, c->n_cu, pr_want, slots, P.rerun, c->d_pairs + 5 * c->pair_cap, c->d_small);
  Params* dp = c->d_params + rp;
  HIP_TRY(hipMemcpyAsync(dp, &P, sizeof(Params), hipMemcpyHostToDevice, stream));
  HIP_TRY(hipEventRecord(c->ev[rp], stream));
  c->ev_used[rp] = true;

  std::vector<Launch> seq;
  launch_sequence(fp, c->n_cu, b->n_pairs, slots, pr_want, &seq);
  hipEvent_t t0 = nullptr, t1 = nullptr;
  if (c->timing) {
    HIP_TRY(take_event(c, &t0));
    HIP_TRY(take_event(c, &t1));
  }
  st = run_sequence(c, seq, dp, stream, !(flags & MICA_NO_GRAPH), t0, t1);
  if (st != MICA_OK) return st;
  if (c->timing) c->ev_pending.emplace_back(t0, t1);
  c->last_pairs = b->n_pairs;
  c->last_slots = (int)slots;
  c->last_scratch = scratch_bytes;
  return MICA_OK;
}

// (for the tests: launch graphs built so far, and held)
void mica_ctx_graphs(mica_ctx_t c, int64_t* built, int64_t* held) {
  *built = c->graph_builds;
  *held = (int64_t)c->graphs.size();
}

mica_status_t mica_ctx_set_timing(mica_ctx_t c, int enable) {
  if (!c) return fail(MICA_ERR_INVALID_ARG, "ctx is NULL");
  c->timing = enable != 0;
  return MICA_OK;
}

mica_status_t mica_ctx_read_timing(mica_ctx_t c, double* fill_ms, int64_t* n_batches) {
  if (!c || !fill_ms || !n_batches) return fail(MICA_ERR_INVALID_ARG, "NULL argument");
  HIP_TRY(hipSetDevice(c->device));
  double total = 0;
  for (auto& pr : c->ev_pending) {
    HIP_TRY(hipEventSynchronize(pr.second));
    float ms = 0;
    HIP_TRY(hipEventElapsedTime(&ms, pr.first, pr.second));
    total += ms;
    c->ev_pool.push_back(pr.first);
    c->ev_pool.push_back(pr.second);
  }
  *fill_ms = total;
  *n_batches = (int64_t)c->ev_pending.size();
  c->ev_pending.clear();
  return MICA_OK;
}

mica_status_t mica_ctx_last_stats(mica_ctx_t c, void* stream, mica_batch_stats_t* out) {
  if (!c || !out) return fail(MICA_ERR_INVALID_ARG, "NULL argument");
  HIP_TRY(hipSetDevice(c->device));
  HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
  uint32_t ctr[kNumCounters];
  HIP_TRY(hipMemcpy(ctr, small_counters(c), sizeof(ctr), hipMemcpyDeviceToHost));
  out->n_pairs = c->last_pairs;
  out->n_items = ctr[kCtrItems];
  out->n_saturated = ctr[kCtrRerun];
  out->n_waves = c->last_slots;
  out->scratch_bytes = (int64_t)c->last_scratch;
  uint32_t fbc[kNumBuckets];
  HIP_TRY(hipMemcpy(fbc, small_fbcount(c), sizeof(fbc), hipMemcpyDeviceToHost));
  out->n_fallback = 0;
  for (int b = 0; b < kNumBuckets; ++b) out->n_fallback += fbc[b];
  out->n_fallback += (int64_t)ctr[kCtrPruneWide] - (int64_t)ctr[kCtrPruneLeft];
  out->n_deferred = ctr[kCtrPruneMid];
  for (size_t list : {small::kDbcount, small::kDbwide}) {
    HIP_TRY(hipMemcpy(fbc, c->d_small + list, sizeof(fbc), hipMemcpyDeviceToHost));
    for (int b = 0; b < kNumBuckets; ++b) out->n_deferred += fbc[b];
  }
  return MICA_OK;
}

}  // extern "C"
