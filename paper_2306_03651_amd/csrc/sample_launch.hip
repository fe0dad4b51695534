// Host side of the single-source path sampler: launch shape, per-BFS slot
// state, the staging area and its redraw on overflow, the layout of the
// staged hyperedges in sample order.  The kernel is in sample.hip.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <string>
#include <utility>
#include <vector>

#include "common.hpp"
#include "internal.hpp"
#include "sample.hpp"

namespace centra {

// Launch shapes: the LDS-bitmap variant runs one 1024-thread workgroup per
// CU (the bitmap takes most of the LDS); the other variants (a 2 KB visited
// filter in LDS) run several workgroups of 64 to 512 threads per CU.
constexpr uint32_t kMaxSlots = 8192;
constexpr uint32_t kLeanSlots = 3072;   // slots beyond which memory is only taken if much is left
constexpr uint32_t kSlotParts = 12;     // 32nds of the device that those may take

// Byte offsets of a launch's counters in work_ctr: the two words that every
// workgroup adds to on lines of their own; then arcs, nodes, entries, and
// the number of deferred items.
constexpr size_t kCtrWork = 0, kCtrUsed = 128, kCtrStats = 256, kCtrBytes = 512;

struct SamplePlan {
  bool lds_bits;
  int block;         // workgroup size of the LDS-filter variants
  uint32_t bit_words;
  size_t dyn_lds;
  uint32_t resident;   // workgroups resident at once = BFS slots
};

// Bytes of one slot's state: per node the map's word, the count and the
// queue entry; the bitmap of level starts; and the pair arrays.
static size_t slot_bytes(uint32_t n) { return size_t(n) * (8 + 8 + 4) + start_words(n) * 8 + kPairMax * 12; }

// Slot state takes at most half of the device's memory (96 GiB if the size
// cannot be queried; asked once per context); the context budget, when set,
// limits it further.
size_t slot_mem_cap(centra_ctx* ctx) {
  if (ctx->slot_cap) return ctx->slot_cap;
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess || total_b == 0) {
    (void)hipGetLastError();
    total_b = size_t(192) << 30;
  }
  return ctx->slot_cap = total_b / 2;
}

// Slots that a launch may have by the rules of memory alone, whatever else is
// allocated.  Up to `lean` of them may take half of the device, or the whole
// budget.  More hide more latency but leave less memory to whatever is
// allocated next, so they may take `parts` 32nds of the device, or an eighth
// of the budget.
static size_t slots_allowed(centra_ctx* ctx, size_t per_slot, uint32_t lean, uint32_t parts) {
  const size_t cap = slot_mem_cap(ctx), most = ctx->budget && ctx->budget < cap ? ctx->budget : cap;
  const size_t room = ctx->budget ? std::min(cap / 16 * parts, ctx->budget / 8) : cap / 16 * parts;
  return std::max(std::min<size_t>(lean, most / per_slot), room / per_slot);
}

// Variant choice.  Default: one wave per BFS where there are many (most BFSs
// are short chains of dependent steps; a wave needs no barrier, and 4,096 of
// them hide each other's trips to memory).  Where there are few, more threads
// each end the longest of them sooner: 256 below 2,048 samples, 128 below
// 32,768.  Where memory holds fewer slots, more threads each use them better:
// 128 below 4,096 slots, 256 below 2,048.  Measured, ms with 64 / 128 / 256
// threads:
//   BA n = 10^6, 1,024 samples: 0.49 / 0.34 / 0.28; 16,384: 1.48 / 1.25 /
//   1.28; 32,768: 2.26 / 2.07 / 2.39; 131,072: 6.2 / 6.9 / 8.7
//   BA n = 10^5, 16,384: 0.52 / 0.54 / 0.71; 65,536: 1.19 / 1.61 / 2.41
//   directed R-MAT scale 20, 16,384: 3.5 / 1.9 / 1.5; 32,768: 4.5 / 2.7 / 2.2
//   BA of more nodes, 200,000 samples, 3,072 slots (64 threads; 128 have
//   2,048, 256 1,024): 18.0 / 16.1 / 19.0; 1,902 slots: 31.6 / 22.3 / 23.3;
//   1,272: 52 / 35 / 29; 955: 74 / 50 / 35
//   directed R-MAT scale 22, 1,814 slots, 500,000 samples: 83 / 53 / 45.
// On small graphs of short rows a level has at most some hundred nodes, and
// one wave each does from 4,096 samples on (kNarrowNodes, kNarrowRow): grid 128
// x 128, 2,048 samples: 3.5 / 3.1 / 3.4, 4,096: 4.2 / 4.7 / 5.6, 16,384: 11.5
// / 13.9 / 17.8; random 4-regular, n = 4,000, 8,192: 0.38 / 0.40 / 0.55.  Not
// on larger graphs (grid 256 x 256, 8,192: 29 / 24 / 28; 4-regular, n = 10^5:
// 4.1 / 3.2 / 2.7) nor with longer rows (16-regular, n = 16,000, 8,192: 0.34 /
// 0.29 / 0.33), be they in-rows alone (8 out-arcs, in-rows of up to 4,484, n =
// 16,000: 2.3 / 1.2 / 0.7).
// A fused or stream-ordered launch leaves no sample for after it, so its
// longest BFS holds it: 128 threads also where the graphs are skewed, which
// long rows tell (fused, directed R-MAT scale 20, 2 x 40,000 samples: 80 / 47 /
// 25; directed, n = 10^5, rows of up to 15,887, 40,000: 29 / 16 / 11; BA n =
// 10^6, rows of up to 3,560, 400,000: 20.0 / 21.6 / 28.1; BA n = 10^5, rows of up
// to 1,134: 7.1 / 10.0 / 15.1; stream-ordered, R-MAT scale 20, 400,000: 68 / 43
// / 26; scale 14, rows of up to 2,443, 40,000: 0.81 / 0.54).
// CENTRA_SAMPLER_VARIANT selects another for single-graph launches: "lds"
// (exact LDS bitmap, 1024 threads, when the bitmap fits), "hbm512", "hbm256",
// "hbm128", "hbm64" (LDS filter, that many threads).
constexpr uint32_t kFewSamples = 2048, kManySamples = 32768, kManyNarrow = 4096;
constexpr uint32_t kNarrowNodes = 32768, kNarrowRow = 8;
constexpr size_t kFewSlots = 2048, kManySlots = 4096;
constexpr uint32_t kSkewedRow = 2048;

// max_row: the longest row of the graph (of a fused launch's graphs) in either
// direction; defers: long BFSs are left for after the launch.
static int threads_for(centra_ctx* ctx, uint32_t n, uint64_t count, uint32_t max_row, bool defers) {
  const size_t slots = slots_allowed(ctx, slot_bytes(n), kLeanSlots, kSlotParts);
  if (slots < kFewSlots || count < kFewSamples) return 256;
  const uint32_t many = n <= kNarrowNodes && max_row <= kNarrowRow ? kManyNarrow : kManySamples;
  return slots < kManySlots || count < many || (!defers && max_row > kSkewedRow) ? 128 : 64;
}

static uint32_t longest_row(const centra_graph* g) { return std::max(g->max_in_degree, g->max_out_degree); }

int fused_threads(centra_ctx* ctx, const MultiSampleItem* items, uint32_t n_items) {
  uint32_t n = 1, max_row = 0;
  for (uint32_t i = 0; i < n_items; ++i) {
    n = std::max(n, items[i].g->n);
    max_row = std::max(max_row, longest_row(items[i].g));
  }
  return threads_for(ctx, n, ~0ull, max_row, false);
}

// multi: a fused launch; block: its threads per BFS if the caller chose them;
// async: a stream-ordered launch.
static SamplePlan plan_for(centra_ctx* ctx, uint32_t n, uint32_t count, uint32_t max_row, bool async,
                           bool multi = false, int block = 0) {
  SamplePlan p{};
  p.bit_words = (n + 31) / 32;
  int max_lds = 0, cus = 0;
  if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, ctx->device) != hipSuccess)
    max_lds = 65536;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess || cus <= 0)
    cus = 256;
  const size_t dyn = size_t(p.bit_words) * 4;
  const char* env = getenv("CENTRA_SAMPLER_VARIANT");
  const char* v = env && !multi ? env : "";
  p.block = block ? block : threads_for(ctx, n, count, max_row, !async && !multi);
  if (!strcmp(v, "hbm64")) p.block = 64;
  if (!strcmp(v, "hbm512")) p.block = 512;
  if (!strcmp(v, "hbm256")) p.block = 256;
  if (!strcmp(v, "hbm128")) p.block = 128;
  p.lds_bits = !strcmp(v, "lds") && sample_lds_variant_bytes() + dyn <= size_t(max_lds);
  int per_cu = 0;
  p.dyn_lds = p.lds_bits ? dyn : 0;
  hipError_t e = sample_kernel_occupancy(p.block, p.lds_bits, multi, p.dyn_lds, &per_cu);
  if (e != hipSuccess || per_cu <= 0) per_cu = 1;
  (void)hipGetLastError();
  const uint64_t r = uint64_t(cus) * uint64_t(per_cu);
  p.resident = r > kMaxSlots ? kMaxSlots : static_cast<uint32_t>(r);
  return p;
}

// Slots for a launch that has a use for `want`, where the state held now
// takes `have` bytes: as many as the rules allow, more than `lean` of them
// only while a quarter of the device remains free (a context that draws from
// both samplers on n = 2 10^6 would otherwise ask for the whole device; with
// three eighths, one on n = 10^6 has 2,700 bidirectional searches at once beside
// the path sampler's state and takes 58.5 ms for 800,000 samples, not 48.2), and
// no more than the budget holds.
uint32_t slots_that_fit(centra_ctx* ctx, size_t per_slot, uint32_t want, uint32_t lean, uint32_t parts, size_t have) {
  const size_t most = std::max<size_t>(1, slots_allowed(ctx, per_slot, lean, parts));
  if (want > most) want = static_cast<uint32_t>(most);
  if (ctx->budget) {
    const size_t others = ctx->allocated - have;
    auto fits = [&](uint32_t slots) { return others + size_t(slots) * per_slot <= ctx->budget; };
    uint32_t slots = want;
    if (!fits(slots))
      for (slots = lean; slots > 1 && !fits(slots);) slots /= 2;
    return slots < want ? slots : want;
  }
  if (want > lean) {
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
      (void)hipGetLastError();
      return lean;
    }
    const size_t keep = slot_mem_cap(ctx) / 2;
    const size_t room = free_b + have > keep ? free_b + have - keep : 0;
    want = std::max<uint32_t>(lean, std::min<size_t>(want, room / per_slot));
  }
  return want;
}

static int ensure_slots(centra_ctx* ctx, uint32_t gn, uint32_t want, hipStream_t s, bool* fresh) {
  *fresh = false;
  // enough of them, or all that this many were cut down to
  if ((ctx->slots >= want && ctx->slot_n >= gn) || (ctx->slot_want >= want && ctx->slot_n == gn)) return CENTRA_OK;
  // a new allocation is sized for this launch alone: keeping the largest n
  // ever seen with the largest slot count ever asked for would grow the
  // state (and its zero fill) to the memory cap after one large graph
  const uint32_t n = gn;
  DevBuf* bufs[] = {&ctx->slot_map, &ctx->slot_sig, &ctx->slot_q, &ctx->slot_starts, &ctx->slot_pinfo};
  size_t have = 0;
  for (DevBuf* b : bufs) have += b->bytes;
  uint32_t slots = slots_that_fit(ctx, slot_bytes(n), want, kLeanSlots, kSlotParts, have);
  if (ctx->slots >= slots && ctx->slot_n >= n) return CENTRA_OK;
  int rc;
  for (;;) {   // halve the slot count while the device cannot hold the state
    for (DevBuf* b : bufs) release(ctx, *b);
    ctx->slots = ctx->slot_want = 0;
    ctx->slot_n = 0;
    rc = ensure(ctx, ctx->slot_map, size_t(slots) * n * 8, false, s);
    if (!rc) rc = ensure(ctx, ctx->slot_sig, size_t(slots) * n * 8, false, s);
    if (!rc) rc = ensure(ctx, ctx->slot_pinfo, size_t(slots) * kPairMax * 12, false, s);
    if (!rc) rc = ensure(ctx, ctx->slot_q, size_t(slots) * n * 4, false, s);
    if (!rc) rc = ensure(ctx, ctx->slot_starts, size_t(slots) * start_words(n) * 8, false, s);
    if (rc != CENTRA_ENOMEM || slots <= 64) break;
    slots /= 2;
  }
  if (rc) return rc;
  fill_u64(static_cast<uint64_t*>(ctx->slot_map.ptr), 0, size_t(slots) * n, s);   // stamp 0: never claimed
  CENTRA_HIP(ctx, hipGetLastError());
  ctx->slots = slots;
  ctx->slot_n = n;
  ctx->slot_want = want;
  *fresh = true;
  return CENTRA_OK;
}

// Deferred samples: a BFS about to expand a level of more than kWideNodes
// nodes, or past the launch's scan budget, is left for after the launch; at
// most kWideCap per launch (the rest finish on their workgroups).  The budget
// is what a workgroup may expect to scan in the whole launch
// (kWideArcsPerItem entries per item of its share): a longer BFS would hold
// the launch after the others have ended.  (Directed R-MAT scale 20, 200,000
// samples, three BFSs of some 2 million entries each: 28.6 ms with the
// largest budget, 14.0 with this one.)
//
// A few of them go through the device-wide BFS (wide_samples in sample.hip),
// which takes the whole GPU for each, 0.2 ms (n = 65,536) to 2.4 (n = 4 10^6),
// so the budget is also at least a share of the graph's arcs (R-MAT scale 22,
// 20,000 samples: 9.2 ms without, 4.0 with; half the share as good, twice as
// much costs scale 20 a ninth).  More of them, of graphs where many BFSs are
// long, are drawn by a second launch with kSecondBlock threads each, from which
// only those past its budget go to the device-wide BFS.  (BA n = 10^6 of 2
// edges per node, 100,000 samples, 1,240 deferred: 1,080 ms all device-wide, 47
// with the second launch, 56 with the largest budget in the first; 256 threads
// in the second launch 49.)
//
// Where both are near, the second launch is a bet: it takes up to 4.5 ns per
// entry of its budget, and gains nothing on floods that end on the device-wide
// BFS all the same (undirected R-MAT scale 18, 100,000 samples, 30 deferred:
// 9.4 ms in vain, the device-wide BFSs 10.3; directed, n = 10^6, long in-rows,
// 25 deferred: 5.4 ms instead of 23.9).  So it is taken where the device-wide
// BFSs would take more than half its time, and may then spend a quarter of
// theirs, or as much as a whole BFS of the graph if that is less than theirs.
constexpr uint32_t kWideNodes = 65536;
constexpr uint64_t kWideArcsPerItem = 4096;
constexpr uint64_t kWideArcsMin = uint64_t(1) << 17, kWideArcsMax = uint64_t(1) << 21;
constexpr uint64_t kWideArcsShare = 128;   // of the graph's arcs
constexpr uint32_t kWideFew = 8;
constexpr int kSecondBlock = 512;
constexpr double kSecondArcMs = 4.5e-6;   // per entry, one BFS
constexpr double kWideMs = 0.2, kWideNodeMs = 0.6e-6;   // per device-wide BFS, and per node of the graph
constexpr uint32_t kWideCap = 4096;
constexpr uint32_t kWideGroup = 64;   // deferred samples advanced together

static bool wide_enabled() {
  const char* e = getenv("CENTRA_WIDE");
  return !(e && !strcmp(e, "0"));
}

// Turns deferral on in `a` (its list, with as much room for the second
// launch's, in ctx->wide_ws, its counter the word after the statistics in
// work_ctr, cleared with them).
static int defer_args(centra_ctx* ctx, SampleArgs& a, uint32_t grid, hipStream_t s) {
  int rc;
  if ((rc = ensure(ctx, ctx->wide_ws, size_t(kWideGroup) * 64 + size_t(kWideCap) * 8, false, s))) return rc;
  a.defer_nodes = kWideNodes;
  a.defer_arcs = std::max({kWideArcsMin, a.n_arcs / kWideArcsShare, a.count / grid * kWideArcsPerItem});
  a.defer_arcs = std::min(kWideArcsMax, a.defer_arcs);
  if (const char* e = getenv("CENTRA_WIDE_NODES")) {   // tests: a lower threshold
    const long v = atol(e);
    if (v >= 1 && v <= 0x7FFFFFFFl) a.defer_nodes = static_cast<uint32_t>(v);
  }
  a.defer_cap = kWideCap;
  a.defer_list = reinterpret_cast<uint32_t*>(static_cast<char*>(ctx->wide_ws.ptr) + size_t(kWideGroup) * 64);
  a.defer_count = reinterpret_cast<uint32_t*>(static_cast<char*>(ctx->work_ctr.ptr) + kCtrStats + 24);
  return CENTRA_OK;
}

// Placement of the slot maps.  How fast the sampler runs depends on where
// the allocator put the pages of the per-BFS node maps: the same launch on
// BA 10^6 varies from one allocation of them to the next (by up to 18% when
// they were 16-byte records), hardly within one, and not when the queues or
// the graph are allocated again.  A short launch ranks allocations as the
// full one does, so fresh maps of at least kPlaceMinBytes are chosen among
// kPlaceCandidates allocations by timing the batch's first kPlaceProbe work
// items on each (second of two launches; results discarded, stamps used up
// as by any launch).  It runs for the context's first large slot state only
// (a context that re-allocates as its graphs change size would pay the
// search each time).  The search holds two map arrays at a time and stops
// early if the budget or the device cannot, or once a step takes more than
// kPlaceStepMs of wall time (slow probes, or freed memory the device must
// clear first); CENTRA_SLOT_SEARCH=0 turns it off.  It synchronises the
// stream, so stream-ordered launches skip it.
constexpr int kPlaceCandidates = 4;
constexpr double kPlaceStepMs = 60.0;   // wall time of one step (allocation, clear, two probes)
constexpr uint32_t kPlaceProbe = 65536;
constexpr size_t kPlaceMinBytes = size_t(4) << 30;

static bool slot_search_enabled() {
  const char* e = getenv("CENTRA_SLOT_SEARCH");
  return !(e && !strcmp(e, "0"));
}

// Sets the per-launch fields of `a` for `count` work items on the current
// slot state and staging area (stage_cap entries).
static void launch_args(centra_ctx* ctx, SampleArgs& a, const SamplePlan& plan, uint32_t count, uint64_t stage_cap,
                        uint32_t stage_chunk) {
  a.stamp0 = ctx->stamp_next;
  ctx->stamp_next += count;
  a.count = count;
  a.slot_stride = ctx->slot_n;
  a.map = static_cast<uint64_t*>(ctx->slot_map.ptr);
  a.sig = static_cast<uint64_t*>(ctx->slot_sig.ptr);
  a.q = static_cast<uint32_t*>(ctx->slot_q.ptr);
  a.starts = static_cast<uint64_t*>(ctx->slot_starts.ptr);
  a.rec = a.sig;   // after the launch, for the device-wide BFS
  a.pinfo = static_cast<uint32_t*>(ctx->slot_pinfo.ptr);
  a.bit_words = plan.bit_words;
  char* ctr = static_cast<char*>(ctx->work_ctr.ptr);
  a.work = reinterpret_cast<uint64_t*>(ctr + kCtrWork);
  a.stats = reinterpret_cast<uint64_t*>(ctr + kCtrStats);
  a.entries = a.stats + 2;
  a.stage_chunk = stage_chunk;
  a.stage = static_cast<uint32_t*>(ctx->stage_nodes.ptr);
  a.stage_cap = stage_cap;
  a.stage_used = reinterpret_cast<uint64_t*>(ctr + kCtrUsed);
  a.stage_pos = static_cast<uint64_t*>(ctx->stage_pos.ptr);
  a.he_len = static_cast<uint32_t*>(ctx->stage_len.ptr);
  a.flags = ctx->d_flags;
  a.defer_nodes = 0;
  a.defer_arcs = 0;
  a.defer_cap = 0;
  a.defer_list = nullptr;
  a.defer_count = nullptr;
  a.items = nullptr;
}

// Stamps: a launch numbers its work items stamp_next, stamp_next + 1, ...;
// before the first launch, and when 32 bits would run out, every map is
// cleared and numbering restarts at 1 (the bidirectional sampler's records
// carry the same stamps).
static void reserve_stamps(centra_ctx* ctx, uint32_t count, hipStream_t s) {
  if (ctx->stamp_next == 0 || uint64_t(ctx->stamp_next) + count > 0xFFFFFFFFull) {
    fill_u64(static_cast<uint64_t*>(ctx->slot_map.ptr), 0, size_t(ctx->slots) * ctx->slot_n, s);
    if (ctx->bi_rec_f.ptr) {
      fill_u64(static_cast<uint64_t*>(ctx->bi_rec_f.ptr), 0, size_t(ctx->bi_slots) * ctx->bi_n * 2, s);
      fill_u64(static_cast<uint64_t*>(ctx->bi_rec_b.ptr), 0, size_t(ctx->bi_slots) * ctx->bi_n * 2, s);
    }
    ctx->stamp_next = 1;
  }
}

// Times two launches of the first `count` work items on the current slot
// state and returns the second's milliseconds in *ms.
static int probe_slots(centra_ctx* ctx, SampleArgs a, const SamplePlan& plan, bool multi, uint32_t count,
                       hipStream_t s, float* ms) {
  for (int rep = 0; rep < 2; ++rep) {
    reserve_stamps(ctx, count, s);
    fill_u64(static_cast<uint64_t*>(ctx->work_ctr.ptr), 0, kCtrBytes / 8, s);
    launch_args(ctx, a, plan, count, ctx->stage_nodes.bytes / 4, kStageChunk);
    // a flooding sample would hold every probe as long as itself: it is
    // left out, as the timed launches leave it to the device-wide BFS
    int rc;
    const uint32_t grid = count < ctx->slots ? count : ctx->slots;
    if (!multi && !plan.lds_bits && wide_enabled() && ctx->slots >= 2 && (rc = defer_args(ctx, a, grid, s))) return rc;
    CENTRA_HIP(ctx, hipEventRecord(ctx->ev[6], s));
    sample_kernel_launch(a, plan.block, plan.lds_bits, multi, grid, plan.dyn_lds, s);
    CENTRA_HIP(ctx, hipGetLastError());
    CENTRA_HIP(ctx, hipEventRecord(ctx->ev[7], s));
    CENTRA_HIP(ctx, hipStreamSynchronize(s));
    if ((rc = check_flags(ctx, s, "sample_paths (placement probe)"))) return rc;
    if (hipEventElapsedTime(ms, ctx->ev[6], ctx->ev[7]) != hipSuccess) *ms = 0.f;
  }
  return CENTRA_OK;
}

// Chooses the fastest of kPlaceCandidates allocations of the (fresh) slot
// maps, by probe_slots.
static int place_slots(centra_ctx* ctx, const SampleArgs& a, const SamplePlan& plan, bool multi, uint32_t count,
                       hipStream_t s) {
  const size_t map_b = ctx->slot_map.bytes;
  if (map_b < kPlaceMinBytes) return CENTRA_OK;
  ctx->placed = true;   // once per context: a later re-allocation keeps what it gets
  const uint32_t pc = count < kPlaceProbe ? count : kPlaceProbe;
  // every slot state held during the search must stay consistent with the
  // stamps: start numbering if nothing has been drawn yet, and skip the
  // search if its launches would run the stamps out (a restart clears only
  // the slot state in use)
  reserve_stamps(ctx, 0, s);
  if (uint64_t(ctx->stamp_next) + uint64_t(2 * kPlaceCandidates) * pc + count > 0xFFFFFFFFull) return CENTRA_OK;
  const auto t0 = std::chrono::steady_clock::now();
  auto since = [](std::chrono::steady_clock::time_point x) {
    return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - x).count();
  };
  float best = 0.f;
  int rc;
  if ((rc = probe_slots(ctx, a, plan, multi, pc, s, &best))) return rc;
  std::string line = "slot placement: " + std::to_string(best);
  // the search stops where it would cost more than it can win: a probe
  // that is slow (long searches) or a step that is (the device clearing
  // freed memory before handing it out again takes seconds for tens of GB)
  bool go = since(t0) <= kPlaceStepMs;
  for (int c = 1; go && c < kPlaceCandidates && best > 0.f; ++c) {
    const auto tc = std::chrono::steady_clock::now();
    if (ctx->budget && ctx->allocated + map_b > ctx->budget) break;
    void* r2 = nullptr;
    if (hipMalloc(&r2, map_b) != hipSuccess) {
      (void)hipGetLastError();
      break;
    }
    fill_u64(static_cast<uint64_t*>(r2), 0, map_b / 8, s);   // stamp 0: never claimed
    std::swap(ctx->slot_map.ptr, r2);
    float ms = 0.f;
    rc = probe_slots(ctx, a, plan, multi, pc, s, &ms);
    line += " " + std::to_string(ms);
    if (rc || !(ms > 0.f && ms < best)) std::swap(ctx->slot_map.ptr, r2);   // keep the previous one
    else best = ms;
    (void)hipStreamSynchronize(s);
    (void)hipFree(r2);
    if (rc) return rc;
    go = since(tc) <= kPlaceStepMs;
  }
  const std::string stop = go ? "" : "; stopped: a step took over " + std::to_string(int(kPlaceStepMs)) + " ms";
  const double took = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  ctx->log += line + " ms -> " + std::to_string(best) + " ms (search " + std::to_string(took) + " ms" + stop + ")\n";
  return CENTRA_OK;
}

// The scan budget of a second launch for n deferred samples of the graph; 0:
// none, they go to the device-wide BFS.
static uint64_t second_budget(const SampleArgs& a, uint32_t n) {
  const double wide = n * (kWideMs + kWideNodeMs * a.n), whole = kSecondArcMs * double(a.n_arcs);
  if (n <= kWideFew || wide <= 0.5 * std::min(whole, kSecondArcMs * double(kWideArcsMax))) return 0;
  if (whole <= wide) return kWideArcsMax;
  return std::min(kWideArcsMax, std::max(kWideArcsMin, static_cast<uint64_t>(0.25 * wide / kSecondArcMs)));
}

// Draws a launch's n deferred samples (in a.defer_list) by a launch of their
// own; what this one defers is in a.defer_list on return (the other half of
// the list).
static int second_launch(centra_ctx* ctx, SampleArgs& a, uint32_t n, uint64_t budget, hipStream_t s) {
  int per_cu = 0, cus = 0;
  if (sample_kernel_occupancy(kSecondBlock, false, false, 0, &per_cu) != hipSuccess || per_cu <= 0) per_cu = 1;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess || cus <= 0)
    cus = 256;
  (void)hipGetLastError();
  const uint32_t grid = std::min(std::min(n, ctx->slots), static_cast<uint32_t>(cus * per_cu));
  reserve_stamps(ctx, n, s);
  a.stamp0 = ctx->stamp_next;
  ctx->stamp_next += n;
  a.count = n;
  a.items = a.defer_list;
  a.defer_list += kWideCap;
  a.defer_arcs = budget;
  a.stage_chunk = 0;
  fill_u64(a.work, 0, 1, s);
  fill_u32(a.defer_count, 0, 1, s);
  CENTRA_HIP(ctx, hipEventRecord(ctx->ev[6], s));
  sample_kernel_launch(a, kSecondBlock, false, false, grid, 0, s);
  CENTRA_HIP(ctx, hipGetLastError());
  CENTRA_HIP(ctx, hipEventRecord(ctx->ev[7], s));
  return CENTRA_OK;
}

// Runs one sampling launch of `count` work items into the staging area
// (redrawn with a larger area if it overflows); `a` holds the graph part of
// the arguments (or the instance table of a fused launch), `max_n` the
// largest n of its graphs, `max_row` their longest row in either direction.
// *total receives the staged node count.
// async_cap != 0: stream-ordered form; the staging area holds async_cap
// entries, the launch is not redrawn, nothing is read back (the caller
// learns the size from the device).
static int launch_sampler(centra_ctx* ctx, SampleArgs a, uint32_t count, uint32_t max_n, uint32_t max_row, bool multi,
                          int block, uint64_t* total, hipStream_t s, uint64_t async_cap = 0) {
  int rc;
  *total = 0;
  const SamplePlan plan = plan_for(ctx, max_n, count, max_row, async_cap != 0, multi, block);
  uint32_t want = count < plan.resident ? count : plan.resident;
  bool fresh = false;
  if ((rc = ensure_slots(ctx, max_n, want, s, &fresh))) return rc;
  // (slots may be left from a launch of more and smaller workgroups)
  const uint32_t grid = want < ctx->slots ? want : ctx->slots;
  if ((rc = ensure(ctx, ctx->stage_pos, size_t(count) * 8, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->stage_len, size_t(count) * 4 + 8 + 8 * (size_t(count) + 1), false, s))) return rc;
  if ((rc = ensure(ctx, ctx->work_ctr, kCtrBytes, false, s))) return rc;
  if (fresh && !ctx->placed && !async_cap && slot_search_enabled() && (rc = place_slots(ctx, a, plan, multi, count, s)))
    return rc;
  // staging: workgroups reserve it in chunks of a few hyperedges of their
  // share, of which each may leave one partly used (a stream-ordered launch's
  // area holds the caller's capacity exactly: there every hyperedge is
  // reserved by itself)
  uint32_t chunk = async_cap ? 0u : std::min(kStageChunk, count / grid * 4);
  const uint64_t slack = uint64_t(grid) * chunk;
  const uint64_t base_cap = async_cap ? async_cap : size_t(count) * 8 + 1024;
  uint64_t cap = base_cap + slack;
  if (!async_cap && ctx->staged_samples) {
    // entries per sample reserved on this context so far, with half again as
    // a margin: an area too small makes the whole launch run twice
    const double per = 1.5 * double(ctx->staged_entries) / double(ctx->staged_samples);
    const uint64_t est = static_cast<uint64_t>(per * double(count)) + 1024 + slack;
    if (est > cap) cap = est;
  }
  if (ctx->stage_nodes.bytes / 4 > cap) cap = ctx->stage_nodes.bytes / 4;
  for (int attempt = 0; attempt < 3; ++attempt) {
    rc = ensure(ctx, ctx->stage_nodes, cap * 4, false, s);
    if (rc == CENTRA_ENOMEM && attempt == 0 && cap > base_cap && ctx->stage_nodes.bytes / 4 < cap) {
      cap = base_cap;   // the estimate does not fit the budget: the plain size, without chunks
      chunk = 0;
      rc = ensure(ctx, ctx->stage_nodes, cap * 4, false, s);
    }
    if (rc == CENTRA_ENOMEM && attempt > 0 && chunk) {   // an exact area, without chunks
      chunk = 0;
      cap -= slack;
      rc = ensure(ctx, ctx->stage_nodes, cap * 4, false, s);
    }
    if (rc) return rc;
    cap = ctx->stage_nodes.bytes / 4;
    fill_u64(static_cast<uint64_t*>(ctx->work_ctr.ptr), 0, kCtrBytes / 8, s);
    reserve_stamps(ctx, count, s);
    launch_args(ctx, a, plan, count, cap, chunk);
    // (a sample's records of the device-wide BFS take two slots' counts)
    const bool wide = !async_cap && !multi && !plan.lds_bits && wide_enabled() && ctx->slots >= 2;
    if (wide && (rc = defer_args(ctx, a, grid, s))) return rc;
    CENTRA_HIP(ctx, hipEventRecord(ctx->ev[6], s));
    sample_kernel_launch(a, plan.block, plan.lds_bits, multi, grid, plan.dyn_lds, s);
    CENTRA_HIP(ctx, hipGetLastError());
    if (async_cap) return CENTRA_OK;
    CENTRA_HIP(ctx, hipEventRecord(ctx->ev[7], s));
    uint64_t ctr[kCtrBytes / 8];
    const uint64_t* stats = ctr + kCtrStats / 8;   // arcs, nodes, entries, deferred
    CENTRA_HIP(ctx, hipMemcpyAsync(ctr, ctx->work_ctr.ptr, kCtrBytes, hipMemcpyDeviceToHost, s));
    CENTRA_HIP(ctx, hipStreamSynchronize(s));
    if ((rc = check_flags(ctx, s, "sample_paths"))) return rc;
    float ms = 0.f, ms2 = 0.f;
    if (hipEventElapsedTime(&ms, ctx->ev[6], ctx->ev[7]) != hipSuccess) ms = 0.f;
    auto deferred = [&]() { return static_cast<uint32_t>(std::min<uint64_t>(stats[3] & 0xFFFFFFFFull, kWideCap)); };
    uint32_t n_wide = wide ? deferred() : 0u;
    if (const uint64_t budget = second_budget(a, n_wide)) {
      if ((rc = second_launch(ctx, a, n_wide, budget, s))) return rc;
      CENTRA_HIP(ctx, hipMemcpyAsync(ctr, ctx->work_ctr.ptr, kCtrBytes, hipMemcpyDeviceToHost, s));
      CENTRA_HIP(ctx, hipStreamSynchronize(s));
      if ((rc = check_flags(ctx, s, "sample_paths (second launch)"))) return rc;
      if (hipEventElapsedTime(&ms2, ctx->ev[6], ctx->ev[7]) != hipSuccess) ms2 = 0.f;
      n_wide = deferred();
    }
    const uint64_t arcs = stats[0], nodes = stats[1];
    if (n_wide) {
      // the deferred samples, one device-wide BFS each, on the slots' queues
      // and (two slots' counts per sample) records
      std::vector<uint32_t> list(n_wide);
      CENTRA_HIP(ctx, hipMemcpyAsync(list.data(), a.defer_list, size_t(n_wide) * 4, hipMemcpyDeviceToHost, s));
      CENTRA_HIP(ctx, hipStreamSynchronize(s));
      uint64_t* ctl = static_cast<uint64_t*>(ctx->wide_ws.ptr);
      std::vector<uint64_t> host_ctl(size_t(kWideGroup) * 8);
      const auto w0 = std::chrono::steady_clock::now();
      const uint32_t group = std::max<uint32_t>(1, std::min<uint32_t>(kWideGroup, ctx->slots / 2));
      for (uint32_t j0 = 0; j0 < n_wide; j0 += group) {   // a group at a time, one slot each
        const uint32_t nj = std::min<uint32_t>(group, n_wide - j0);
        uint64_t wide_arcs = 0;
        if (wide_samples(a, list.data() + j0, nj, ctl, host_ctl.data(), &wide_arcs, s) != CENTRA_OK)
          return hip_fail(ctx, hipGetLastError(), "sample_paths (device-wide BFS)");
        ctx->st.wide_arcs += wide_arcs;
      }
      ctx->st.wide_ms += std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - w0).count();
      CENTRA_HIP(ctx, hipMemcpyAsync(ctr, ctx->work_ctr.ptr, kCtrBytes, hipMemcpyDeviceToHost, s));
      CENTRA_HIP(ctx, hipStreamSynchronize(s));
      if ((rc = check_flags(ctx, s, "sample_paths (device-wide BFS)"))) return rc;
      ctx->st.wide += n_wide;
    }
    const uint64_t used = ctr[kCtrUsed / 8], entries = stats[2];
    ctx->st.launches += 1;
    ctx->st.kernel_ms += ms + ms2;
    ctx->st.samples += count;
    ctx->st.arcs += arcs;
    ctx->st.nodes += nodes;
    ctx->st.hyperedge_nodes += used <= cap ? entries : 0;
    ctx->st.lds_bitmap = plan.lds_bits ? 1 : 0;
    ctx->st.slots = grid;
    if (used <= cap) {
      *total = entries;
      ctx->staged_entries += used;
      ctx->staged_samples += count;
      return CENTRA_OK;
    }
    cap = used + slack + 1024;   // staging overflowed: the batch is redrawn identically
  }
  return fail(ctx, CENTRA_EHIP, "sample_paths: staging did not converge");
}

int sample_to_stage(centra_ctx* ctx, const centra_graph* g, uint64_t seed, uint32_t instance, uint64_t first,
                    uint32_t count, uint32_t* st_out, uint32_t* dist_out, uint64_t* total, hipStream_t s) {
  *total = 0;
  if (count == 0) return CENTRA_OK;
  SampleArgs a{};
  a.n = g->n;
  a.n_arcs = g->n_arcs;
  a.c_bits = g->count_bits;
  a.max_out_deg = g->max_out_degree;
  a.row_ptr = g->bfs_row_ptr;
  a.col_idx = g->bfs_col_idx;
  a.in_ptr = g->bfs_in_ptr;
  a.in_idx = g->bfs_in_idx;
  a.new_of = g->new_of;
  a.orig_of = g->orig_of;
  a.seed = seed;
  a.instance = instance;
  a.first = first;
  a.st_out = st_out;
  a.dist_out = dist_out;
  return launch_sampler(ctx, a, count, g->n, longest_row(g), false, 0, total, s);
}

int sample_multi_to_stage(centra_ctx* ctx, const MultiSampleItem* items, uint32_t n_items, int block,
                          uint64_t* total, hipStream_t s) {
  *total = 0;
  std::vector<SampleInst> tab;
  std::vector<uint32_t> off;
  uint64_t count = 0;
  uint32_t max_n = 0, max_row = 0;
  for (uint32_t i = 0; i < n_items; ++i) {
    const MultiSampleItem& it = items[i];
    if (it.count == 0) continue;
    const centra_graph* g = it.g;
    SampleInst x{};
    x.n = g->n;
    x.c_bits = g->count_bits;
    x.max_out_deg = g->max_out_degree;
    x.instance = it.instance;
    x.row_ptr = g->bfs_row_ptr;
    x.col_idx = g->bfs_col_idx;
    x.in_ptr = g->bfs_in_ptr;
    x.in_idx = g->bfs_in_idx;
    x.new_of = g->new_of;
    x.orig_of = g->orig_of;
    x.seed = it.seed;
    x.first = it.first;
    tab.push_back(x);
    off.push_back(static_cast<uint32_t>(count));
    count += it.count;
    max_n = std::max(max_n, g->n);
    max_row = std::max(max_row, longest_row(g));
  }
  if (count == 0) return CENTRA_OK;
  if (count >= (1ull << 32)) return fail(ctx, CENTRA_ENOTSUP, "sample_multi: 2^32 work items or more");
  off.push_back(static_cast<uint32_t>(count));
  int rc;
  const size_t tab_bytes = tab.size() * sizeof(SampleInst);
  if ((rc = ensure(ctx, ctx->multi_tab, tab_bytes + off.size() * 4 + 256, false, s))) return rc;
  char* dtab = static_cast<char*>(ctx->multi_tab.ptr);
  const size_t off_at = (tab_bytes + 255) & ~size_t(255);
  CENTRA_HIP(ctx, hipMemcpyAsync(dtab, tab.data(), tab_bytes, hipMemcpyHostToDevice, s));
  CENTRA_HIP(ctx, hipMemcpyAsync(dtab + off_at, off.data(), off.size() * 4, hipMemcpyHostToDevice, s));
  SampleArgs a{};
  a.inst = reinterpret_cast<const SampleInst*>(dtab);
  a.item_off = reinterpret_cast<const uint32_t*>(dtab + off_at);
  a.n_inst = static_cast<uint32_t>(tab.size());
  rc = launch_sampler(ctx, a, static_cast<uint32_t>(count), max_n, max_row, true, block, total, s);
  CENTRA_HIP(ctx, hipStreamSynchronize(s));   // the host tables above go out of scope
  return rc;
}

// Lays staged hyperedges out after the base = he_off[0] entries already in
// the store: he_off[i] = base + rel[i] and the nodes at he_nodes + base +
// rel[i] when end = base + rel[count] fits `cap`; otherwise every new
// hyperedge is stored empty (he_off[i] = base, nothing beyond the store
// is referenced) and kErrCapacity is raised.  *total = end either way.
// he_off[0] (rel[0] = 0) is read by every thread and written by none.
__global__ void k_stage_append(uint32_t count, const uint64_t* stage_pos, const uint32_t* he_len, const uint64_t* rel,
                               const uint32_t* stage, uint64_t* he_off, uint32_t* he_nodes, uint64_t cap,
                               uint64_t* total, uint32_t* flags) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i > count) return;
  const uint64_t base = he_off[0];
  const uint64_t end = base + rel[count];
  const bool fits = end <= cap;
  if (i > 0) he_off[i] = fits ? base + rel[i] : base;
  if (i == count) {
    if (total) *total = end;
    if (!fits) atomicOr(flags, kErrCapacity);
    return;
  }
  if (!fits) return;
  const uint64_t p = stage_pos[i];
  const uint64_t o = base + rel[i];
  const uint32_t len = he_len[i];
  for (uint32_t x = 0; x < len; ++x) he_nodes[o + x] = stage[p + x];
}

int sample_reserve(centra_ctx* ctx, const centra_graph* g, uint32_t count, uint64_t stage_entries, hipStream_t s) {
  const SamplePlan plan = plan_for(ctx, g->n, count, longest_row(g), true);
  const uint32_t want = count < plan.resident ? count : plan.resident;
  int rc;
  bool fresh = false;   // no placement search here: there is no launch to time
  if ((rc = ensure_slots(ctx, g->n, want ? want : 1, s, &fresh))) return rc;
  if ((rc = ensure(ctx, ctx->stage_pos, size_t(count) * 8, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->stage_len, size_t(count) * 4 + 8 + 8 * (size_t(count) + 1), false, s))) return rc;
  if ((rc = ensure(ctx, ctx->work_ctr, kCtrBytes, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->stage_nodes, (stage_entries ? stage_entries : 1) * 4, false, s))) return rc;
  return ensure(ctx, ctx->scan_tmp, scan_tile_words(count) * 8, false, s);
}

int sample_append(centra_ctx* ctx, const centra_graph* g, uint64_t seed, uint32_t instance, uint64_t first,
                  uint32_t count, uint64_t* he_off, uint32_t* he_nodes, uint64_t he_cap, uint64_t* he_total,
                  hipStream_t s) {
  if (count == 0) return CENTRA_OK;
  SampleArgs a{};
  a.n = g->n;
  a.n_arcs = g->n_arcs;
  a.c_bits = g->count_bits;
  a.max_out_deg = g->max_out_degree;
  a.row_ptr = g->bfs_row_ptr;
  a.col_idx = g->bfs_col_idx;
  a.in_ptr = g->bfs_in_ptr;
  a.in_idx = g->bfs_in_idx;
  a.new_of = g->new_of;
  a.orig_of = g->orig_of;
  a.seed = seed;
  a.instance = instance;
  a.first = first;
  uint64_t total = 0;
  int rc = launch_sampler(ctx, a, count, g->n, longest_row(g), false, 0, &total, s, he_cap ? he_cap : 1);
  if (rc) return rc;
  uint32_t* len = static_cast<uint32_t*>(ctx->stage_len.ptr);
  uint64_t* rel = reinterpret_cast<uint64_t*>(static_cast<char*>(ctx->stage_len.ptr) + ((size_t(count) * 4 + 7) & ~size_t(7)));
  if ((rc = excl_scan_u32_to_u64(ctx, len, rel, count, s))) return rc;
  hipLaunchKernelGGL(k_stage_append, dim3((count + 1 + 255) / 256), dim3(256), 0, s, count,
                     static_cast<const uint64_t*>(ctx->stage_pos.ptr), len, rel,
                     static_cast<const uint32_t*>(ctx->stage_nodes.ptr), he_off, he_nodes, he_cap, he_total,
                     ctx->d_flags);
  CENTRA_HIP(ctx, hipGetLastError());
  return CENTRA_OK;
}

int stage_to_output(centra_ctx* ctx, uint32_t count, uint64_t base, uint64_t* he_off, uint32_t* he_nodes,
                    hipStream_t s) {
  uint32_t* len = static_cast<uint32_t*>(ctx->stage_len.ptr);
  uint64_t* rel = reinterpret_cast<uint64_t*>(static_cast<char*>(ctx->stage_len.ptr) + ((size_t(count) * 4 + 7) & ~size_t(7)));
  int rc = excl_scan_u32_to_u64(ctx, len, rel, count, s);
  if (rc) return rc;
  stage_gather_launch(count, static_cast<const uint64_t*>(ctx->stage_pos.ptr), len, rel, base,
                      static_cast<const uint32_t*>(ctx->stage_nodes.ptr), he_off, he_nodes, s);
  CENTRA_HIP(ctx, hipGetLastError());
  return CENTRA_OK;
}

}  // namespace centra
