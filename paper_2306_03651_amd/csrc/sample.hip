// sampleHEs for set betweenness on gfx950.
//
// Each workgroup of a persistent grid owns one BFS slot and takes sample
// indices from an atomic work counter until the batch is exhausted.  One
// sample = pair draw, level-synchronous BFS from s with normalised path
// counts, backtrack of a uniform shortest path from t.  Every quantity the
// output depends on (levels, integer count sums, level maxima, the ordered
// scan of in-neighbours) is independent of thread timing, so the result is
// bit-identical to a sequential implementation.
//
// State of a slot, in HBM: the visited nodes in level order (their ids and
// counts sigma', contiguous), a bitmap of the places where levels start, and a
// map from nodes to places in that order (Visited, below): one 8-byte word per node, stamp
// << 32 | place, where the stamp numbers the BFSs of the context in launch
// and work order.  A slot's map carries only stamps older than its current
// BFS's unless that BFS visited the node, so nothing is ever reset between
// samples (the map starts at stamp 0; the stamps restart after a full clear
// when 32 bits run out).  An LDS filter holds the visited nodes.
//
// Level expansion (push): the frontier is processed in chunks of BLOCK
// nodes, whose arcs are spread evenly over the workgroup (ArcSpread).  An
// arc w -> v that finds v's filter bit clear claims v, with its own
// contribution; the others go to a table of duplicates in LDS (Dups), which
// sums them per node and looks the nodes up together.  The largest raw count
// of the level, which decides the normalisation shift, comes from the counts
// as they are written, so it needs no extra pass; only when the shift is
// nonzero are the level's counts rewritten.
//
// What bounds it: a BFS is a chain of dependent trips to memory (about 60
// at BA n = 10^6, of 0.5 to 2 us), and with 4,096 of them in flight the
// waves' instructions (a SIMD issues in 79% of its cycles).  So the kernel
// uses no global atomic in a BFS, looks nodes up in bulk (Hits, Dups), and
// keeps its code within the instruction cache (41 KB of 64; 83 KB before,
// when every launch and most steps waited for instructions).  Measured, with
// 16-byte records claimed by returning 64-bit global atomics before, from one
// box and placement of the state to another: BA n = 10^6, 400,000 samples,
// 26.7-31 -> 15.2-17.6 ms; grid 128 x 128, 10,000 samples, 13.9-14.4 ->
// 7.7-8.2 ms; directed R-MAT scale 20, 200,000 samples, 32-49 -> 14.3 ms (21 while
// all deferred samples went one after another through the device-wide BFS).
//
// Early stop.  After levels 0..L are complete, every visited in-neighbour
// of an unvisited node is at level L (a lower one would have put the node
// in a completed level).  Before expanding level L the workgroup tests, on
// rings of in-neighbours around t:
//   (1) t has a visited in-neighbour: d(s,t) = L+1;
//   (2) some pair (w in in(t), u in in(w)) has u visited: w is at L+1 and
//       d = L+2; the raw count of each such w is the sum of its visited
//       in-neighbours' counts;
//   (3) some u of those pairs (unvisited) has visited in-neighbours: u is
//       at L+1, its w at L+2 and d = L+3; the raw counts of u and w follow
//       the same way (the test sums them per w; the backtrack counts again
//       the u of the one w it picks).
// Levels L+1 (and L+2) are then never produced.  Their normalisation
// would be a no-op when every count of theirs is below 2^C: level L+1
// counts are at most S_L (the sum of the level-L counts) and level L+2
// counts at most S_L times the largest out-degree, so (2) is taken only if
// S_L < 2^C and (3) only if also S_L * max out-degree < 2^C; otherwise the
// levels are produced and normalised as usual.  Test (3) scans the in-rows
// of the ring's nodes (the cone), so it runs only when the cone is at most
// kConeRatio times the CSR entries that expanding level L would scan, and
// (2) only when its pairs are at most kPairRatio times those entries.  All
// routes give the same counts, hence the same hyperedge.
//
// Unreachable targets.  A t without in-neighbours skips the BFS; when the
// rings show that every ancestor of t is within backward distance 1 or 2,
// the BFS stops once the tests have ruled out those distances.
//
// Node ids.  The kernel traverses the graph's locality-relabelled copy
// (grouped so that nodes reached from one hub have nearby ids); the pair
// is drawn in caller ids and mapped in, and hyperedge nodes are mapped back.
// Rows keep the caller's order, so every scan order is the caller's.
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "common.hpp"
#include "internal.hpp"
#include "sample.hpp"

namespace centra {

// Ring limits: t with at most Ring<BLOCK>::kCache in-neighbours gets the
// 2-hop test on the pairs (w in in(t), u in in(w)); the 3-hop test also
// needs at most kPairMax pairs.  Cost rules (kConeRatio, kPairRatio) decide
// at which levels they run.
template <int BLOCK>
struct Ring {
  static constexpr uint32_t kCache = BLOCK >= 512 ? 512u : BLOCK >= 128 ? 256u : 128u;
};
// Bits of the visited filter (see Visited).
constexpr uint32_t kBitLog = 14;
constexpr uint32_t kBitWords = (1u << kBitLog) / 32;
constexpr uint64_t kConeRatio = 3;
// The 2-hop test runs at a level only when its pairs are at most kPairRatio
// times the out-arcs expanding that level would scan (2 and 4 measure alike,
// 1 is 2% slower; of cone ratios 1, 2, 3, 4 and 6, 1 is 40% slower, 2 4%).
constexpr uint64_t kPairRatio = 4;

// Entries a round handles per thread (loads in flight), and in all: the
// duplicate table and the hit lists below hold a round's.
template <int BLOCK>
struct Round {
  static constexpr int kPer = BLOCK <= 128 ? 4 : BLOCK <= 512 ? 2 : 1;
  static constexpr uint32_t kArcs = BLOCK * kPer;
  // slots of the duplicate table: twice a round's arcs where LDS allows it
  // without a workgroup less per CU
  static constexpr uint32_t kSlots = BLOCK == 128 ? kArcs + kArcs / 2 : BLOCK == 256 || BLOCK == 512 ? 2 * kArcs : kArcs;
  static constexpr int kMasks = kArcs / kWave;   // <= 64: one per lane
};

template <int BLOCK>
struct SampleShared {
  uint64_t sg[BLOCK];                    // per source of a chunk: its count, its ring index, or the sum of its arcs
  uint64_t ring[Ring<BLOCK>::kCache];    // per in-neighbour w of t: its count on the level the last test gave it
  uint64_t dsum[Round<BLOCK>::kSlots];   // duplicate table: sums (zero when empty); in the tests the waves' hit lists
  uint64_t mask[3][Round<BLOCK>::kMasks];   // arcs of a round that start a source's run
  uint64_t red[2 * Coll<BLOCK>::kHalf];
  uint64_t hub_pairs;
  uint64_t pk_weight;                    // the entry a pick chose: its weight,
  uint32_t pk[4];                        // index, node and in-row bounds
  uint32_t dkey[Round<BLOCK>::kSlots];   // duplicate table: nodes, kUnseen when empty
  uint32_t rs[BLOCK];                    // per source of a chunk: row start less the arcs before it
  uint32_t fr[BLOCK];                    // the first nodes of the newest level
  uint32_t poff[Ring<BLOCK>::kCache];    // pair offsets of t's in-neighbours
  uint32_t rrs[Ring<BLOCK>::kCache];     // in_ptr[w] less that offset: pair p's entry is in_idx[rrs + p]
  uint32_t bits[BLOCK >= 1024 ? 1 : kBitWords];   // visited filter (the 1024-thread variant's is dynamic)
  uint32_t hpos;
  uint32_t pick;
  uint32_t qlen;
  uint32_t next;
};

// Visited set of one BFS.  Visited nodes are numbered in queue order; node
// v's place is map[v], valid if it carries the BFS's stamp, and its count is
// sig[place].  So a claim is one scattered 8-byte store (and two stores at
// the end of the queue), the level of a node is where its place lies among
// the level starts, and only the map is spread over the n nodes.
//
// An LDS filter holds every claimed node: a clear bit proves that a node is
// unvisited without touching memory.  A node's bit is its id modulo the
// filter's size: exact where n fits it (the 1024-thread variant's dynamic
// bitmap, or n up to 2^kBitLog).  Setting a node's bit with
// a returning LDS atomic claims the node if the bit was clear: of all arcs
// that reach it one sees the bit clear.  No global atomic takes part in a
// BFS: they are all carried out at the memory side here, past the L2 (as
// many EA atomics as L2 atomics were counted), at about 2 us each.
struct Visited {
  uint32_t* bits;       // LDS
  uint32_t mask;        // bit of node v: v & mask
  bool exact;
  uint64_t* map;
  const uint32_t* q;
  uint64_t* sig;
  uint64_t base;        // the BFS's stamp << 32

  __device__ __forceinline__ uint32_t bit(uint32_t v) const { return v & mask; }
  __device__ __forceinline__ bool maybe(uint32_t v) const {
    const uint32_t b = bit(v);
    return (bits[b >> 5] >> (v & 31u)) & 1u;
  }
  // sets v's bit; true if it was clear
  __device__ __forceinline__ bool set(uint32_t v) const {
    const uint32_t b = bit(v), m = 1u << (v & 31u);
    return !(atomicOr(&bits[b >> 5], m) & m);
  }
  // v's place, kUnseen if v is not visited
  __device__ __forceinline__ uint32_t place(uint32_t v) const {
    const uint64_t e = wg_ld_u64(&map[v]) - base;
    return e < kUnseen ? static_cast<uint32_t>(e) : kUnseen;
  }
  __device__ __forceinline__ bool visited(uint32_t v) const { return maybe(v) && (exact || place(v) != kUnseen); }
  // sigma'_v of a visited v, else 0 (between levels every claimed node is on
  // a completed one)
  __device__ __forceinline__ uint64_t count(uint32_t v) const {
    if (!maybe(v)) return 0;
    const uint32_t p = place(v);
    return p != kUnseen ? wg_ld_u64(&sig[p]) : 0ull;
  }
};

// Arcs of a chunk of sources, one source per thread, spread over the
// workgroup.  The sources with arcs are numbered in thread order; source c
// holds arcs [off_c, off_c + deg_c) of the chunk.  A round takes kArcs
// consecutive arcs, arc base + k * BLOCK + tid in a thread's chain k, and
// marks in a bit mask (in LDS) the arcs that are a source's first: an arc's
// source is then the number of marks at or before it, less one, which a
// wave reads off one mask word with a popcount of the marks before.  (A
// binary search of the offsets takes log2(BLOCK) dependent LDS reads per
// arc; it was most of the instructions of a level.)  The masks of three
// rounds are held in turn: a round zeroes the one that the round after the
// next will use.
template <int BLOCK>
struct ArcSpread {
  SampleShared<BLOCK>& sh;
  uint32_t turn;     // the mask of the coming round
  uint32_t before;   // sources that start before the coming round

  // every mask zero, before the first chunk (a barrier must follow)
  __device__ __forceinline__ void init() {
    for (int i = threadIdx.x; i < 3 * Round<BLOCK>::kMasks; i += BLOCK) (&sh.mask[0][0])[i] = 0;
    turn = 0;
  }
  // marks source start `off` if it lies in the round of arcs from base
  __device__ __forceinline__ void mark(bool has, uint32_t off, uint32_t base) {
    const uint32_t o = off - base;
    if (has && off >= base && o < Round<BLOCK>::kArcs)
      atomicOr(reinterpret_cast<unsigned long long*>(&sh.mask[turn][o >> 6]), 1ull << (o & 63u));
  }
  // the round's sources: src[k] of the thread's arc k (meaningful for arcs
  // below the chunk's total).  A barrier lies between mark and this.
  __device__ __forceinline__ void sources(uint32_t (&src)[Round<BLOCK>::kPer]) {
    constexpr int NM = Round<BLOCK>::kMasks;
    const int lane = lane_id();
    const uint32_t wid = uniform_u32(threadIdx.x / kWave);
    const uint64_t m = lane < NM ? sh.mask[turn][lane] : 0ull;
    const uint32_t clear = turn == 0 ? 2u : turn - 1u;
    if (threadIdx.x < NM) sh.mask[clear][threadIdx.x] = 0;
    turn = turn == 2 ? 0u : turn + 1u;
    const uint32_t pc = static_cast<uint32_t>(__popcll(m));
    const uint32_t incl = wave_incl_scan_u32(pc);
    const uint32_t excl = incl - pc;
#pragma unroll
    for (int k = 0; k < Round<BLOCK>::kPer; ++k) {
      const int w = static_cast<int>(k * (BLOCK / kWave) + wid);
      // marks before this word, and of the word at or below the lane (its
      // bit 0, and of the rest shifted down those below the lane)
      const uint64_t mk = lane_u64(m, w);
      const uint32_t at = before + lane_u32(excl, w) + static_cast<uint32_t>(mk & 1ull) - 1u;
      const uint32_t lo = static_cast<uint32_t>(mk >> 1), hi = static_cast<uint32_t>(mk >> 33);
      src[k] = at + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
    }
    before += lane_u32(incl, kWave - 1);
  }
};

// Nodes whose filter bit is set, met in a scan between levels, with the index
// in `into` of the sum they count for: that of the row's source (kDirect),
// or the one sh.sg names for it.  Looking a node up takes two
// dependent trips to memory (its place, its count), so a wave collects the
// nodes of many rounds in its share of the duplicate table's sums and looks
// them up together, all loads in flight.
template <int BLOCK, bool kDirect>
struct Hits {
  static constexpr int PER = Round<BLOCK>::kPer;
  static constexpr uint32_t kCap = PER * kWave;   // entries per wave: a round's at least
  SampleShared<BLOCK>& sh;
  const Visited& vis;
  uint64_t* into;   // LDS
  uint64_t* list;   // this wave's
  uint32_t n;       // entries (uniform over the wave)
  bool any;         // a listed node was visited

  __device__ __forceinline__ Hits(SampleShared<BLOCK>& sh_, const Visited& vis_, uint64_t* into_)
      : sh(sh_), vis(vis_), into(into_), list(sh_.dsum + uniform_u32(threadIdx.x / kWave) * kCap), n(0), any(false) {}
  // Adds the round's nodes x[k] (kUnseen: none) of the rows of sources
  // src[k]; looks the listed nodes up if these no longer fit, or if it is the
  // last round (which may be empty).  Every lane calls.
  __device__ __forceinline__ void round(const uint32_t (&x)[PER], const uint32_t (&src)[PER], bool last) {
    uint64_t m[PER];
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      m[k] = __ballot(x[k] != kUnseen && vis.maybe(x[k]));
      c += static_cast<uint32_t>(__popcll(m[k]));
    }
    for (;;) {
      if (n + c > kCap || (last && c == 0 && n)) {
        uint32_t p[PER], r[PER];
        uint64_t w[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          const uint32_t i = k * kWave + lane_id();
          p[k] = kUnseen;
          r[k] = 0;
          if (i < n) {
            const uint64_t e = list[i];
            list[i] = 0;
            r[k] = static_cast<uint32_t>(e);
            p[k] = vis.place(static_cast<uint32_t>(e >> 32));
          }
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) w[k] = p[k] != kUnseen ? wg_ld_u64(&vis.sig[p[k]]) : 0ull;
#pragma unroll
        for (int k = 0; k < PER; ++k)
          if (w[k]) {   // (a produced count is never 0)
            any = true;
            atomicAdd(reinterpret_cast<unsigned long long*>(&into[r[k]]), static_cast<unsigned long long>(w[k]));
          }
        n = 0;
      }
      if (c == 0) break;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        if ((m[k] >> lane_id()) & 1ull)
          list[n + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m[k] >> 32),
                                             __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m[k]), 0))] =
              uint64_t(x[k]) << 32 | (kDirect ? src[k] : static_cast<uint32_t>(sh.sg[src[k]]));
        n += static_cast<uint32_t>(__popcll(m[k]));
      }
      c = 0;
      if (!last) break;
    }
  }
};

// Raw counts of one chunk of unvisited nodes, one per thread with its in-row
// (start rs_u, length deg; 0 for none): returns the sum of sigma' over the
// node's visited in-neighbours.  Every one of them is at the last produced
// level (a lower one would have put the node in a produced level), so this
// is the node's raw count one level below.  Contains barriers.
template <int BLOCK>
__device__ __forceinline__ uint64_t raw_counts_chunk(const uint32_t* in_idx, const Visited& vis, uint32_t rs_u,
                                                     uint32_t deg, SampleShared<BLOCK>& sh, Coll<BLOCK>& co,
                                                     ArcSpread<BLOCK>& sp) {
  constexpr int PER = Round<BLOCK>::kPer;
  constexpr uint32_t R = BLOCK * PER;
  const uint32_t tid = threadIdx.x;
  uint32_t off, c, total;
  co.scan_and_rank(deg, &off, &c, &total);
  if (total == 0) return 0;   // uniform
  if (deg) {
    sh.rs[c] = rs_u - off;
    sh.sg[c] = 0;
  }
  sp.before = 0;
  Hits<BLOCK, true> hits(sh, vis, sh.sg);
  for (uint32_t base = 0; base < total; base += R) {
    sp.mark(deg != 0, off, base);
    __syncthreads();
    uint32_t x[PER], j[PER];
    sp.sources(j);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const uint32_t e = base + k * BLOCK + tid;
      x[k] = kUnseen;
      if (e < total) x[k] = in_idx[sh.rs[j[k]] + e];
    }
    hits.round(x, j, base + R >= total);
  }
  __syncthreads();
  // (sg is written again only after the next chunk's scan, which has a barrier)
  return deg ? sh.sg[c] : 0ull;
}

// Weighted pick over entries j = 0 .. len-1 in ascending order, workgroup
// wide: W = sum of the weights (or W_known when nonzero, the caller's exact
// sum), r = bounded(st, W), and the result is the smallest j whose
// inclusive prefix sum exceeds r; kUnseen when W = 0.  Each thread holds
// kPickPer consecutive entries per round, so a round covers BLOCK *
// kPickPer entries with that many loads in flight; rows of at most one
// round are summed and searched from the same registers.  load(j0, cnt, w)
// fills w[0 .. cnt) for entries j0 on (cnt <= kPickPer, all at once); the
// one thread that holds the pick calls chosen(k, j, weight), for its entry
// k of the round, and what it leaves in LDS is there for every thread on
// return.  Uniform control flow; every thread draws the same words.
constexpr uint32_t kPickPer = 4;

template <int BLOCK, typename Load, typename Chosen>
__device__ __forceinline__ uint32_t block_pick(uint32_t len, const Load& load, const Chosen& chosen, uint64_t W_known,
                                               RolledWordStream& st, SampleShared<BLOCK>& sh, Coll<BLOCK>& co) {
  constexpr uint32_t kRound = BLOCK * kPickPer;
  const uint32_t first = threadIdx.x * kPickPer;
  uint64_t x[kPickPer];
  uint64_t W = W_known, run = 0, r = 0;
  // sum the row first if it is longer than a round and its sum is unknown
  bool summing = len > kRound && !W;
  if (W) r = bounded(st, W);
  for (uint32_t c = 0; c < len;) {
    const uint32_t j0 = c + first;
    const uint32_t cnt = j0 < len ? (len - j0 < kPickPer ? len - j0 : kPickPer) : 0u;
#pragma unroll
    for (uint32_t k = 0; k < kPickPer; ++k) x[k] = 0;
    load(j0, cnt, x);
    uint64_t ts = 0, tot;
#pragma unroll
    for (uint32_t k = 0; k < kPickPer; ++k) ts += x[k];
    uint64_t excl = run + co.scan(ts, &tot);
    c += kRound;
    if (!W && (!summing || c >= len)) {   // the sum is complete: draw
      W = run + tot;
      if (!W) return kUnseen;
      r = bounded(st, W);
      if (summing) {   // search the row from its start
        summing = false;
        c = 0;
        run = 0;
        continue;
      }
    }
    if (!summing && run + tot > r) {
      if (excl <= r && r < excl + ts) {
#pragma unroll
        for (uint32_t k = 0; k < kPickPer; ++k) {
          if (excl <= r && r < excl + x[k]) {
            sh.pk[0] = j0 + k;
            chosen(k, j0 + k, x[k]);
          }
          excl += x[k];
        }
      }
      __syncthreads();
      return uniform_u32(sh.pk[0]);
    }
    run += tot;
  }
  return kUnseen;
}

__device__ __forceinline__ uint32_t caller_id(const SampleArgs& a, uint32_t v) { return a.orig_of ? a.orig_of[v] : v; }

// A BFS past its scan budget is handed over only on a level of at least
// this many nodes or arcs (a few hubs hold millions): the device-wide BFS
// pays a host round trip per level, so deep, narrow searches (long grids)
// stay on their workgroups.
constexpr uint32_t kWideMinWidth = 4096;
constexpr uint64_t kWideMinArcs = 65536;

// Appends sample idx to the deferred list (workgroup uniform); true if
// it fit, the sample then being left for after the launch.
template <int BLOCK>
__device__ __forceinline__ bool defer_sample(const SampleArgs& a, uint32_t idx, SampleShared<BLOCK>& sh) {
  if (threadIdx.x == 0) {
    const uint32_t at = atomicAdd(a.defer_count, 1u);
    if (at < a.defer_cap) a.defer_list[at] = idx;
    sh.pick = at;
  }
  __syncthreads();
  const uint32_t at = uniform_u32(sh.pick);
  __syncthreads();
  return at < a.defer_cap;
}

// One graph and sample stream, as a work item sees them.
struct GraphArgs {
  uint32_t n, c_bits, max_out_deg, instance;
  const uint32_t* row_ptr;
  const uint32_t* col_idx;
  const uint32_t* in_ptr;
  const uint32_t* in_idx;
  const uint32_t* new_of;
  const uint32_t* orig_of;
  uint64_t seed, first;
};
// Cost rule of the hub 2-hop test at a level (queue entries [lb, le)):
// true when the in-rows of t's dt in-neighbours (starting at in_idx[tb])
// hold at most kPairRatio times the out-arcs of the level.  Both sums grow
// chunk by chunk only until the comparison is decided; the in-row sum and
// its position persist in sh across levels.  Uniform; contains barriers.
template <int BLOCK>
__device__ __forceinline__ bool hub_rule(const GraphArgs& g, const uint32_t* q, uint32_t tb, uint32_t dt, uint32_t lb,
                                      uint32_t le, SampleShared<BLOCK>& sh, Coll<BLOCK>& co, uint64_t& n_arcs) {
  const uint32_t tid = threadIdx.x;
  uint32_t hpos = uniform_u32(sh.hpos);
  uint64_t hub = uniform_u64(sh.hub_pairs);
  uint32_t fpos = lb;
  uint64_t fpart = 0;
  bool run;
  for (;;) {
    const bool hdone = hpos >= dt, fdone = fpos >= le;
    if (hdone && hub <= kPairRatio * fpart) {
      run = true;
      break;
    }
    if (fdone && hub > kPairRatio * fpart) {
      run = false;
      break;
    }
    if (!hdone && (fdone || hub <= kPairRatio * fpart)) {
      const uint32_t e = hpos + tid;
      uint64_t c = 0;
      if (e < dt) {
        const uint32_t w = g.in_idx[tb + e];
        c = g.in_ptr[w + 1] - g.in_ptr[w];
      }
      hub += co.sum(c);
      n_arcs += dt - hpos < uint32_t(BLOCK) ? dt - hpos : uint32_t(BLOCK);
      hpos += BLOCK;
    } else {
      const uint32_t i = fpos + tid;
      uint64_t c = 0;
      if (i < le) {
        const uint32_t w = wg_ld_u32(&q[i]);
        c = g.row_ptr[w + 1] - g.row_ptr[w];
      }
      fpart += co.sum(c);
      fpos += BLOCK;
    }
  }
  __syncthreads();
  if (tid == 0) {
    sh.hpos = hpos;
    sh.hub_pairs = hub;
  }
  __syncthreads();
  return run;
}

// Ring index of pair p: largest i with poff[i] <= p.
__device__ __forceinline__ int ring_of(const uint32_t* poff, uint32_t dt, uint32_t p) {
  int lo = 0, hi = static_cast<int>(dt) - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (poff[mid] <= p)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Appends the wave's newly claimed nodes to the queue: their places follow
// one LDS atomic per wave (none in a workgroup of one wave, whose queue
// length qn is a register).  Returns the thread's place.
template <int BLOCK>
__device__ __forceinline__ uint32_t append(bool has, uint32_t v, uint32_t le, const Visited& vis, uint32_t* q,
                                           SampleShared<BLOCK>& sh, uint32_t& qn) {
  const uint64_t m = __ballot(has);
  if (!m) return 0;   // uniform over the wave
  uint32_t at;
  if constexpr (BLOCK == kWave) {
    at = qn;
    qn += static_cast<uint32_t>(__popcll(m));
  } else {
    uint32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(&sh.qlen, static_cast<uint32_t>(__popcll(m)));
    at = uniform_u32(base);
  }
  at += __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                  __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0));
  if (has) {
    wg_st_u64(&vis.map[v], vis.base | at);
    wg_st_u32(&q[at], v);
    if (at - le < uint32_t(BLOCK)) sh.fr[at - le] = v;
  }
  return at;
}

// Arcs of an expansion whose target's bit was already set.  Each reaches a
// node of a completed level (dropped), a node of the level being produced
// (its contribution is added), or an unvisited node whose bit another node
// set (claimed now).  Their contributions are summed per node in an LDS hash
// table, and a look-up takes every node of the table, all loads in flight
// together: one thread per node then adds the sum or claims the node, so no
// global atomic is needed, and the two trips to memory of a look-up are paid
// per table, not per round.  A workgroup of one wave fills the table over
// several rounds; with more waves it is looked up after every round, by the
// threads that entered the nodes.
//
// In a flood nearly every arc is such a one, so the table must not fill up:
// of a table with no more slots than a round has arcs the last entries take
// hundreds of probes each, and those were most of a flooding BFS's time
// (directed, n = 10^5, 8 out-arcs each, long in-rows, 20,000 samples, all on
// their workgroups: 64 threads 33.7 -> 16.8 ms, 128 22.3 -> 10.2, 256 19.6 ->
// 5.9, 512 12.1 -> 4.7).
template <int BLOCK>
struct Dups {
  static constexpr uint32_t kSlots = Round<BLOCK>::kSlots;
  static constexpr int PER = Round<BLOCK>::kPer;
  SampleShared<BLOCK>& sh;
  const Visited& vis;
  uint32_t n;   // nodes in the table (workgroups of one wave)

  // Nodes v[k] with places p[k] (0: none) and sums x[k]: adds the sum to the
  // count of a node of the new level, claims an unvisited one with it.
  template <int N>
  __device__ __forceinline__ void settle(const uint32_t (&v)[N], const uint32_t (&p)[N], const uint64_t (&x)[N],
                                         uint32_t le, uint32_t* q, uint32_t& qn, uint64_t& mx, uint64_t& added) {
    uint64_t old[N];
#pragma unroll
    for (int k = 0; k < N; ++k) old[k] = p[k] >= le && p[k] != kUnseen ? wg_ld_u64(&vis.sig[p[k]]) : 0ull;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const bool claims = p[k] == kUnseen;
      const uint32_t at = append<BLOCK>(claims, v[k], le, vis, q, sh, qn);
      if (p[k] >= le) {   // (completed levels and empty slots lie below)
        added = sat_add(added, x[k]);
        const uint64_t c = old[k] + x[k];
        wg_st_u64(&vis.sig[claims ? at : p[k]], c);
        mx = c > mx ? c : mx;
      }
    }
    __syncthreads();   // the table is empty, the counts are in place
  }
  // Adds c for node v; true if it was not in the table, *slot its place there.
  // (A round enters at most as many nodes as the table has slots, so a free
  // one is found.)
  __device__ __forceinline__ bool put(uint32_t v, uint64_t c, uint32_t* slot = nullptr) {
    uint32_t h = static_cast<uint32_t>(uint64_t(v * 0x9E3779B1u) * kSlots >> 32);
    uint32_t was;
    for (;;) {
      was = atomicCAS(&sh.dkey[h], kUnseen, v);
      if (was == kUnseen || was == v) break;
      h = (h + 1) % kSlots;
    }
    atomicAdd(reinterpret_cast<unsigned long long*>(&sh.dsum[h]), static_cast<unsigned long long>(c));
    if (slot) *slot = h;
    return was == kUnseen;
  }
  // One wave: looks the table's nodes up and empties it.
  __device__ __forceinline__ void flush(uint32_t le, uint32_t* q, uint32_t& qn, uint64_t& mx, uint64_t& added) {
    constexpr int kOwn = kSlots / BLOCK;
    __syncthreads();   // the entries and the new nodes are in place
    uint32_t v[kOwn], p[kOwn];
    uint64_t x[kOwn];
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const uint32_t i = k * BLOCK + threadIdx.x;
      v[k] = sh.dkey[i];
      x[k] = sh.dsum[i];
      sh.dkey[i] = kUnseen;
      sh.dsum[i] = 0;
      p[k] = v[k] != kUnseen ? vis.place(v[k]) : 0u;
    }
    n = 0;
    settle(v, p, x, le, q, qn, mx, added);
  }
  // Several waves: a round's arcs (bit k of dup set, node v[k] with
  // contribution c[k]) entered and looked up.
  __device__ __forceinline__ void round(uint32_t dup, const uint32_t (&v)[PER], const uint64_t (&c)[PER], uint32_t le,
                                        uint32_t* q, uint32_t& qn, uint64_t& mx, uint64_t& added) {
    uint32_t i[PER], p[PER];
    uint64_t x[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (!((dup >> k) & 1u) || !put(v[k], c[k], &i[k])) i[k] = kUnseen;
    __syncthreads();   // the entries and the new nodes are in place
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      p[k] = 0;
      x[k] = 0;
      if (i[k] == kUnseen) continue;
      x[k] = sh.dsum[i[k]];
      sh.dkey[i[k]] = kUnseen;
      sh.dsum[i[k]] = 0;
      p[k] = vis.place(v[k]);
    }
    settle(v, p, x, le, q, qn, mx, added);
  }
};

// The last level start before place `end` (> 0), a place of the level before
// the one that starts there: the highest set bit below it, 64 words a step.
__device__ __forceinline__ uint32_t last_start(const uint64_t* starts, uint32_t end) {
  const uint32_t last = (end - 1) >> 6;
  for (uint32_t w0 = last;; w0 -= kWave) {   // (bit 0 is set: level 0 starts there)
    const uint32_t lane = lane_id();
    uint64_t x = lane <= w0 ? wg_ld_u64(&starts[w0 - lane]) : 0ull;
    if (w0 - lane == last) x &= ~0ull >> (63u - ((end - 1) & 63u));
    const uint64_t m = __ballot(x != 0);
    if (m) {
      const int l = __ffsll(static_cast<unsigned long long>(m)) - 1;
      return (w0 - l) * 64 + 63 - static_cast<uint32_t>(__clzll(lane_u64(x, l)));
    }
  }
}

// Work items a workgroup takes at once while more than kTakeWhile per
// workgroup are left (then one at a time, to end together).
constexpr uint32_t kTake = 4, kTakeWhile = 16;

// The instance table is not written during a launch: read through the
// constant address space it comes by scalar loads.
using ConstInst = const SampleInst __attribute__((address_space(4)))*;

// Up to 512 threads the kernel is held to 4 waves per SIMD (128 VGPRs): at 5
// it spills 40 registers and is slower (BA n = 10^6: 16.3 against 15.5 ms).
//
// MULTI: a fused launch over several graphs (sample pools).  Each work
// item's graph is looked up in the instance table; every other step is the
// same, so each hyperedge equals that of a launch on its graph alone.
template <int BLOCK, bool LDS_BITS, bool MULTI = false>
__global__ __launch_bounds__(BLOCK, BLOCK <= 512 ? 4 : 1) void k_sample_paths(SampleArgs a) {
  constexpr int PER = Round<BLOCK>::kPer;
  constexpr uint32_t R = Round<BLOCK>::kArcs;   // arcs of an expansion round
  __shared__ SampleShared<BLOCK> sh;
  extern __shared__ uint32_t dyn_bits[];
  const uint32_t tid = threadIdx.x;
  const int lane = lane_id();
  const size_t slot = blockIdx.x;
  uint32_t* q = a.q + slot * a.slot_stride;
  uint64_t* starts = a.starts + slot * start_words(a.slot_stride);
  uint32_t* pu = a.pinfo + slot * 3 * kPairMax;   // per pair: u, in_ptr[u], in-degree of u
  uint32_t* prs = pu + kPairMax;
  uint32_t* pdg = prs + kPairMax;
  Visited vis{};
  vis.bits = LDS_BITS ? dyn_bits : sh.bits;
  vis.mask = LDS_BITS ? ~0u : (1u << kBitLog) - 1u;
  vis.map = a.map + slot * a.slot_stride;
  vis.q = q;
  vis.sig = a.sig + slot * a.slot_stride;
  Coll<BLOCK> co{sh.red, 0};
  ArcSpread<BLOCK> sp{sh, 0, 0};
  sp.init();
  for (uint32_t i = tid; i < Round<BLOCK>::kSlots; i += BLOCK) {
    sh.dkey[i] = kUnseen;
    sh.dsum[i] = 0;
  }
  if (LDS_BITS)
    for (uint32_t i = tid; i < a.bit_words; i += BLOCK) dyn_bits[i] = 0;
  // work counters (uniform across the workgroup): arcs scanned, nodes
  // visited, hyperedge entries staged
  uint64_t n_arcs = 0, n_nodes = 0, n_entries = 0;
  // the rest of the workgroup's chunk of the staging area (thread 0)
  uint64_t st_pos = 0;
  uint32_t st_left = 0;

  // Work items: the first is the workgroup's own number, later ones come
  // from the counter, kTake at a time while many are left (every workgroup
  // adds to the one word, at the memory side).
  uint32_t idx = blockIdx.x, in_hand = 1;
  uint32_t inst_lo = 0, inst_beg = 0, inst_end = 0;   // fused launches: the item's instance and its items
  while (idx < a.count) {
    GraphArgs g;
    if constexpr (MULTI) {
      // the instance of work item idx: the last j with item_off[j] <= idx;
      // 64 candidates a step, and none while the instance stays the same
      if (idx < inst_beg || idx >= inst_end) {
        uint32_t lo = 0, size = a.n_inst;
        while (size > 1) {
          const uint32_t step = (size + kWave - 1) / kWave;
          const uint32_t j = lo + static_cast<uint32_t>(lane) * step;
          const uint64_t m = __ballot(j < lo + size && a.item_off[j < lo + size ? j : lo] <= idx);
          const uint32_t s = 63u - static_cast<uint32_t>(__clzll(m));   // lane 0 always holds
          size = lo + size - (lo + s * step) < step ? lo + size - (lo + s * step) : step;
          lo += s * step;
        }
        inst_lo = uniform_u32(lo);
        inst_beg = uniform_u32(a.item_off[inst_lo]);
        inst_end = uniform_u32(a.item_off[inst_lo + 1]);
      }
      const ConstInst ip = reinterpret_cast<ConstInst>(reinterpret_cast<uintptr_t>(a.inst)) + inst_lo;
      g.n = ip->n;
      g.c_bits = ip->c_bits;
      g.max_out_deg = ip->max_out_deg;
      g.instance = ip->instance;
      g.row_ptr = ip->row_ptr;
      g.col_idx = ip->col_idx;
      g.in_ptr = ip->in_ptr;
      g.in_idx = ip->in_idx;
      g.new_of = ip->new_of;
      g.orig_of = ip->orig_of;
      g.seed = ip->seed;
      g.first = ip->first - inst_beg;   // sample = first + idx (mod 2^64)
    } else {
      g = GraphArgs{a.n, a.c_bits, a.max_out_deg, a.instance, a.row_ptr, a.col_idx, a.in_ptr,
                    a.in_idx, a.new_of, a.orig_of, a.seed, a.first};
    }
    const uint64_t cap = g.c_bits >= 64 ? ~0ull : (1ull << g.c_bits);
    // the sample's place in the batch (a second launch draws listed ones)
    uint32_t out = idx;
    if constexpr (!LDS_BITS && !MULTI) {
      if (a.items) out = uniform_u32(a.items[idx]);
    }
    const uint64_t sample = g.first + out;
    vis.base = uint64_t(a.stamp0 + idx) << 32;
    vis.exact = LDS_BITS || g.n <= (1u << kBitLog);

    // pair draw: every thread draws the same words (uniform, no broadcast)
    RolledWordStream st(g.seed, sample, g.instance, 0);
    const uint32_t s0 = static_cast<uint32_t>(bounded(st, g.n));
    const uint32_t tp = static_cast<uint32_t>(bounded(st, g.n - 1));
    const uint32_t t0 = tp + (tp >= s0 ? 1u : 0u);
    const uint32_t s = g.new_of ? g.new_of[s0] : s0;   // traversal ids
    const uint32_t t = g.new_of ? g.new_of[t0] : t0;

    if constexpr (!LDS_BITS) {
      // the filter starts with s alone
      const uint32_t sb = vis.bit(s);
      for (uint32_t i = tid; i < kBitWords; i += BLOCK) sh.bits[i] = i == sb >> 5 ? 1u << (sb & 31u) : 0u;
    }
    if (tid == 0) {
      wg_st_u64(&vis.map[s], vis.base);
      wg_st_u64(&vis.sig[0], 1);
      wg_st_u32(&q[0], s);
      wg_st_u64(&starts[0], 1);
      sh.fr[0] = s;
      if (LDS_BITS) (void)vis.set(s);
      sh.qlen = 1;
    }

    // Rings around t: R1 = in(t), the pairs (w in R1, u in in(w)) and, if
    // the cone is small enough, in(u) for those u.  poff[i] = number of
    // pairs before R1's i-th entry.  The cone's size (CSR entries a 3-hop
    // test scans) is summed lazily: pairs [0, cpos) so far.
    const uint32_t tb = g.in_ptr[t], te = g.in_ptr[t + 1];
    const uint32_t dt = te - tb;
    const bool rings = dt <= Ring<BLOCK>::kCache;
    uint32_t pairs = 0, cpos = 0;
    uint64_t cone_part = 0;
    uint32_t tw = kUnseen;   // this thread's in-neighbour of t (when they fit the workgroup)
    if (rings) {
      for (uint32_t cb = 0; cb < dt; cb += BLOCK) {
        const uint32_t i = cb + tid;
        uint32_t dw = 0, r0 = 0;
        if (i < dt) {
          const uint32_t w = g.in_idx[tb + i];
          if (cb == 0) tw = w;
          r0 = g.in_ptr[w];
          dw = g.in_ptr[w + 1] - r0;
        }
        uint64_t tot;
        const uint32_t o = pairs + static_cast<uint32_t>(co.scan(dw, &tot));
        if (i < dt) {
          sh.poff[i] = o;
          sh.rrs[i] = r0 - o;
          sh.ring[i] = 0;
        }
        pairs += static_cast<uint32_t>(tot);
      }
      n_arcs += dt;
    }
    __syncthreads();
    // sizes the cone over the next pairs, kConeStep per thread, keeping each
    // pair's u and in-row for the 3-hop test
    constexpr uint32_t kConeStep = 4;
    auto cone_step = [&]() {
      uint32_t u[kConeStep], r0[kConeStep], r1[kConeStep];
      uint64_t dg = 0;
#pragma unroll
      for (uint32_t k = 0; k < kConeStep; ++k) {
        const uint32_t p = cpos + k * BLOCK + tid;
        u[k] = kUnseen;
        if (p < pairs) u[k] = g.in_idx[sh.rrs[ring_of(sh.poff, dt, p)] + p];
      }
#pragma unroll
      for (uint32_t k = 0; k < kConeStep; ++k) {
        r0[k] = u[k] != kUnseen ? g.in_ptr[u[k]] : 0u;
        r1[k] = u[k] != kUnseen ? g.in_ptr[u[k] + 1] : 0u;
      }
#pragma unroll
      for (uint32_t k = 0; k < kConeStep; ++k) {
        const uint32_t p = cpos + k * BLOCK + tid;
        if (p < pairs) {
          dg += r1[k] - r0[k];
          if (p < kPairMax) {
            wg_st_u32(&pu[p], u[k]);
            wg_st_u32(&prs[p], r0[k]);
            wg_st_u32(&pdg[p], r1[k] - r0[k]);
          }
        }
      }
      cone_part += co.sum(dg);
      n_arcs += pairs - cpos < kConeStep * BLOCK ? pairs - cpos : kConeStep * BLOCK;
      cpos += kConeStep * BLOCK;
    };
    // Depth of t's ancestors when the rings show it: every ancestor of t is
    // within backward distance `depth`, so a reachable t has d <= depth and
    // the BFS can stop once the tests have ruled out d <= depth.  Pairs = 0
    // (t's in-neighbours have no in-neighbours) gives 1; a cone of size 0
    // gives 2 (sized here only when the pairs fit one chunk).
    uint32_t depth = kUnseen;
    if (rings && dt) {
      if (pairs == 0) {
        depth = 1;
      } else if (pairs <= BLOCK) {
        cone_step();
        if (cone_part == 0) depth = 2;
      }
    }

    // Row i of `rows` (start, length; none past the end): the in-row of pair
    // i's u, kept by cone_step, or of t's i-th in-neighbour w.
    auto row_of = [&](bool cone, uint32_t i, uint32_t rows, uint32_t* r0, uint32_t* dg) {
      *r0 = 0;
      *dg = 0;
      if (i >= rows) return;
      if (cone) {
        *r0 = wg_ld_u32(&prs[i]);
        *dg = wg_ld_u32(&pdg[i]);
      } else if (rings) {
        const uint32_t o = sh.poff[i];
        *r0 = sh.rrs[i] + o;
        *dg = (i + 1 < dt ? sh.poff[i + 1] : pairs) - o;
      } else {
        const uint32_t w = g.in_idx[tb + i];
        *r0 = g.in_ptr[w];
        *dg = g.in_ptr[w + 1] - *r0;
      }
    };

    // The 2-hop test of a t with more in-neighbours than the ring cache
    // scans the in-rows of all of them (sh.hub_pairs entries, sized lazily
    // over in(t) entries [0, sh.hpos); kept in LDS, as they are read once
    // per level); like test (2) it runs at a level only when those entries
    // are at most kPairRatio times the out-arcs expanding the level would
    // scan.
    if (tid == 0) {
      sh.hpos = 0;
      sh.hub_pairs = 0;
      if (!rings) sh.ring[0] = 0;
    }
    if (!rings) __syncthreads();   // hpos is read at the first level
    uint32_t lb = 0, le = 1, L = 0, d = kUnseen;
    uint32_t qn = 1;          // queue length (workgroups of one wave; else sh.qlen)
    uint64_t sumL = 1;        // S_L: sum of the level-L counts (saturating)
    uint32_t shortcut = 0;    // 2 or 3: levels L+1 (and L+2) were not produced
    uint64_t shifted = 0;     // bit l: the counts of produced level l < 64 were shifted
    // t without in-neighbours is unreachable: no BFS at all (on skewed
    // directed graphs such targets are common, and s may reach millions)
    bool deferred = false, ended = false;
    const uint64_t arcs0 = n_arcs;   // this BFS's scans are n_arcs - arcs0
    for (; dt != 0;) {
      // (1) a visited in-neighbour of t: it is at level L (an earlier check
      //     would have fired otherwise), so d = L + 1
      bool found = false;
      n_arcs += dt;
      if (rings && dt <= BLOCK) {
        found = tid < dt && vis.visited(tw);
      } else {
        for (uint32_t e = tb + tid; e < te; e += BLOCK)
          if (vis.visited(g.in_idx[e])) found = true;
      }
      if (co.any(found)) {
        d = L + 1;
        break;
      }
      if (L + 1 >= depth) break;   // every d <= depth ruled out: unreachable
      // the level's first nodes (from LDS) and their out-rows: the cost
      // rules and the expansion share them
      uint32_t f_w = 0, f_rs = 0, f_deg = 0;
      if (tid < le - lb) {
        f_w = sh.fr[tid];
        f_rs = g.row_ptr[f_w];
        f_deg = g.row_ptr[f_w + 1] - f_rs;
      }
      // out-arcs of level L (the cost of expanding it), summed in workgroup
      // chunks only as far as a cost rule below needs: most produced levels
      // are never expanded
      uint32_t fpos = lb;
      uint64_t fpart = 0;
      auto fcost_step = [&]() {
        uint32_t c = f_deg;
        if (fpos != lb) {
          const uint32_t i = fpos + tid;
          c = 0;
          if (i < le) {
            const uint32_t w = wg_ld_u32(&q[i]);
            c = g.row_ptr[w + 1] - g.row_ptr[w];
          }
        }
        fpart += co.sum(c);
        fpos += BLOCK;
      };
      // tests (2) and (3): each scans rows for visited entries
      for (uint32_t hop = 2; hop <= 3; ++hop) {
        uint32_t rows = 0;
        if (hop == 3) {
          // (3) cone: an unvisited u with visited in-neighbours is at L+1
          //     (they are all at L), its w at L+2 and d = L+3.  Only when
          //     the counts of levels L+1 and L+2 cannot need a shift (level
          //     L+1 counts <= S_L, level L+2 counts <= S_{L+1} <= S_L * max
          //     out-degree) and when the cone is at most kConeRatio times
          //     the out-arcs of level L.  That comparison grows both sums
          //     chunk by chunk until it is decided; sizing the cone also
          //     keeps each pair's u and in-row for the test.  No u is
          //     visited: test (2) has just ruled it out.
          if (!rings || pairs > kPairMax) break;
          const uint64_t bound = (g.max_out_deg && sumL > ~0ull / g.max_out_deg) ? ~0ull : sumL * g.max_out_deg;
          if (sumL >= cap || bound >= cap) break;
          for (;;) {
            const bool cdone = cpos >= pairs, fdone = fpos >= le;
            if (cdone && cone_part <= kConeRatio * fpart) {
              rows = pairs;
              break;
            }
            if (fdone && cone_part > kConeRatio * fpart) break;
            if (!cdone && (fdone || cone_part <= kConeRatio * fpart))
              cone_step();
            else
              fcost_step();
          }
        } else if (rings) {
          // (2) pairs (w, u), the in-rows of t's in-neighbours: a visited u
          //     is at level L (w is unvisited, so a lower level would have
          //     put w in a produced level), hence w at L+1 and d = L+2;
          //     ring[i] = sum of sigma'_u over visited u, the raw count of
          //     w_i (all zero before: set up so, and a test that hits
          //     without ending the BFS clears it)
          const uint64_t need2 = (pairs + kPairRatio - 1) / kPairRatio;
          while (fpos < le && fpart < need2) fcost_step();
          if (fpart >= need2) rows = dt;
        } else if (sumL < cap && hub_rule<BLOCK>(g, q, tb, dt, lb, le, sh, co, n_arcs)) {
          // the same for a t with more in-neighbours than the ring cache
          // (their counts are summed in ring[0])
          rows = dt;
        }
        if (!rows) break;
        Hits<BLOCK, false> hits(sh, vis, sh.ring);
        const bool cone = hop == 3;
        uint32_t r0, dg;
        row_of(cone, tid, rows, &r0, &dg);
        for (uint32_t cb = 0; cb < rows; cb += BLOCK) {
          const uint32_t deg = dg, rs = r0;
          row_of(cone, cb + BLOCK + tid, rows, &r0, &dg);   // on its way meanwhile
          uint32_t off, c, total;
          co.scan_and_rank(deg, &off, &c, &total);
          n_arcs += total;
          if (deg) {
            sh.rs[c] = rs - off;
            sh.sg[c] = cone ? ring_of(sh.poff, dt, cb + tid) : rings ? cb + tid : 0u;
          }
          sp.before = 0;
          const bool last = cb + BLOCK >= rows;
          for (uint32_t base = 0; base < total || last; base += R) {
            sp.mark(deg != 0, off, base);
            __syncthreads();
            uint32_t x[PER], j[PER];
            sp.sources(j);
#pragma unroll
            for (int k = 0; k < PER; ++k) {
              const uint32_t e = base + k * BLOCK + tid;
              x[k] = kUnseen;
              if (e < total) x[k] = g.in_idx[sh.rs[j[k]] + e];
            }
            const bool end = last && base + R >= total;
            hits.round(x, j, end);
            if (end) break;
          }
        }
        if (co.any(hits.any)) {
          if (cone || sumL < cap) {
            // no count of level L+1 can need a shift (each <= S_L < 2^C)
            d = L + hop;
            shortcut = hop;
          } else {
            for (uint32_t i = tid; i < dt; i += BLOCK) sh.ring[i] = 0;
          }
          break;
        }
        if (L + hop >= depth) {   // every d <= depth ruled out: unreachable
          ended = true;
          break;
        }
      }
      if (shortcut || ended) break;
      if constexpr (!LDS_BITS && !MULTI) {
        // a level too wide for one workgroup, or a wide level of a BFS past
        // the scan budget: the sample is deferred (if the list has room) and
        // redrawn in full after the launch
        if (a.defer_nodes &&
            (le - lb > a.defer_nodes || (n_arcs - arcs0 > a.defer_arcs && le - lb >= kWideMinWidth)) &&
            defer_sample<BLOCK>(a, out, sh)) {
          deferred = true;
          break;
        }
      }
      // expand level L (queue entries [lb, le)) into level L+1
      const uint32_t nl = L + 1;
      uint64_t mx = 0, added = 0;
      Dups<BLOCK> dups{sh, vis, 0};
      // rounds of R arcs, chunk of BLOCK frontier nodes after chunk: a
      // round's targets are loaded while the round before is worked on
      uint32_t cb = lb, base = 0, total = 0, off = 0, deg = 0;
      uint64_t lvl_arcs = 0;   // arcs of the level's chunks so far
      uint32_t v[PER];
      uint64_t add[PER];
      for (bool first = true;; first = false) {
        bool more = base < total;
        if (!more && cb < le) {   // the next chunk
          const uint32_t i = cb + tid;
          uint32_t rs = f_rs;
          uint64_t sw = 0;
          deg = 0;
          if (i < le) {
            deg = f_deg;
            if (cb != lb) {
              const uint32_t w = wg_ld_u32(&q[i]);
              rs = g.row_ptr[w];
              deg = g.row_ptr[w + 1] - rs;
            }
            sw = wg_ld_u64(&vis.sig[i]);
          }
          uint32_t c;
          co.scan_and_rank(deg, &off, &c, &total);
          n_arcs += total;
          if (deg) {
            sh.rs[c] = rs - off;
            sh.sg[c] = sw;
          }
          sp.before = 0;
          base = 0;
          cb += BLOCK;
          more = true;   // (a round of no arcs if the chunk has none)
          if constexpr (!LDS_BITS && !MULTI) {
            // a level whose arcs run past the scan budget (hub frontiers): the
            // sample is deferred (uniform; the partial level is abandoned with
            // the BFS's stamp)
            lvl_arcs += total;
            if (a.defer_nodes && n_arcs - arcs0 > a.defer_arcs &&
                (le - lb >= kWideMinWidth || lvl_arcs >= kWideMinArcs) && defer_sample<BLOCK>(a, out, sh)) {
              deferred = true;
              more = false;
            }
          }
        }
        uint32_t nv[PER];
        uint64_t nadd[PER];
        if (more) {
          sp.mark(deg != 0, off, base);
          __syncthreads();
          uint32_t j[PER];
          sp.sources(j);
#pragma unroll
          for (int k = 0; k < PER; ++k) {
            const uint32_t e = base + k * BLOCK + tid;
            nv[k] = 0;
            nadd[k] = 0;
            if (e < total) {
              nv[k] = g.col_idx[sh.rs[j[k]] + e];
              nadd[k] = sh.sg[j[k]];
            }
          }
          base += R;
        }
        uint32_t dup = 0, n_dup = 0;   // bit k: arc k's target had its bit set
        if (!first) {
#pragma unroll
          for (int k = 0; k < PER; ++k) {
            // a node whose bit was clear is new, with this arc's count
            const bool arc = add[k] != 0;   // (a produced count is never 0)
            const bool fresh = arc && vis.set(v[k]);
            const uint32_t at = append<BLOCK>(fresh, v[k], le, vis, q, sh, qn);
            if (fresh) {
              wg_st_u64(&vis.sig[at], add[k]);
              mx = add[k] > mx ? add[k] : mx;
              added = sat_add(added, add[k]);
            }
            const bool again = arc && !fresh;
            if (again) dup |= 1u << k;
            if (BLOCK == kWave) n_dup += static_cast<uint32_t>(__popcll(__ballot(again)));
          }
        }
        if constexpr (BLOCK == kWave) {
          // the table is looked up before more than kMost of its slots would
          // be taken, and at the level's end; a round that alone would take
          // more goes in two halves
          constexpr uint32_t kMost = Round<BLOCK>::kSlots - Round<BLOCK>::kSlots / 8;
          const bool many = n_dup > kMost;
          const uint32_t later = many ? dup >> (PER / 2) << (PER / 2) : 0u;
          dup ^= later;
          for (bool flush = dups.n && dups.n + n_dup > kMost, half = many;;) {
            if (flush) dups.flush(le, q, qn, mx, added);
            bool entered[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) entered[k] = ((dup >> k) & 1u) && dups.put(v[k], add[k]);
#pragma unroll
            for (int k = 0; k < PER; ++k) dups.n += static_cast<uint32_t>(__popcll(__ballot(entered[k])));
            dup = half ? later : 0u;
            if (!half && !(!more && dups.n)) break;
            half = false;
            flush = true;
          }
        } else if (!first) {
          dups.round(dup, v, add, le, q, qn, mx, added);
        }
        if (!more) break;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          v[k] = nv[k];
          add[k] = nadd[k];
        }
      }
      if (deferred) break;   // uniform
      // level L+1 is complete: its largest raw count decides the shift;
      // S_{L+1} is the sum of the added contributions, or of the shifted
      // counts when a shift applies (the collective's barrier closes the
      // level: its queue entries, counts and filter bits are in place)
      co.max_and_sat_sum(&mx, &added);
      const uint32_t ne = BLOCK == kWave ? qn : uniform_u32(sh.qlen);
      if (ne == le) break;   // nothing new: t unreachable
      const uint32_t bl = bitlen64(mx);
      const uint32_t shift = bl > g.c_bits ? bl - g.c_bits : 0u;
      sumL = added;
      // the new level's words of the start bitmap: its first place's bit, the
      // earlier levels' below it, none above
      for (uint32_t w = (le >> 6) + tid; w <= (ne - 1) >> 6; w += BLOCK) {
        uint64_t x = 0;
        if (w == le >> 6) {
          const uint64_t bit = 1ull << (le & 63u);
          x = bit | (le & 63u ? wg_ld_u64(&starts[w]) & (bit - 1) : 0ull);
        }
        wg_st_u64(&starts[w], x);
      }
      if (shift) {
        uint64_t ssum = 0;
        for (uint32_t i = le + tid; i < ne; i += BLOCK) {
          uint64_t x = wg_ld_u64(&vis.sig[i]) >> shift;
          x = x ? x : 1ull;
          wg_st_u64(&vis.sig[i], x);
          ssum = sat_add(ssum, x);
        }
        sumL = co.sat_sum(ssum);
        __syncthreads();   // the level's counts are in place
        if (nl < 64) shifted |= 1ull << nl;
      }
      lb = le;
      le = ne;
      L = nl;
    }

    // (a deferred sample stages nothing here)
    if (!deferred) {
      // backtrack: from v = t, pick a predecessor w at level(v) - 1 with
      // probability sigma'_w / W, scanning in-neighbours in ascending order,
      // until level 1.  Workgroup wide (block_pick); steps through unproduced
      // levels (shortcut 2 or 3) take their weights from the ring sums and the
      // stored pair counts.
      const uint32_t len = (d != kUnseen && d >= 2) ? d - 1 : 0u;
      // the place of the hyperedge in the staging area: only thread 0 writes
      // there.  It takes places from a chunk of its workgroup's (one add on
      // the shared word per chunk); a hyperedge of more than half a chunk
      // gets its own.
      uint64_t hbase = 0;
      if (tid == 0 && len) {
        if (len <= st_left) {
          hbase = st_pos;
          st_pos += len;
          st_left -= len;
        } else if (2 * len > a.stage_chunk) {
          hbase = atomicAdd(reinterpret_cast<unsigned long long*>(a.stage_used), static_cast<unsigned long long>(len));
        } else {
          hbase = atomicAdd(reinterpret_cast<unsigned long long*>(a.stage_used),
                            static_cast<unsigned long long>(a.stage_chunk));
          st_pos = hbase + len;
          st_left = a.stage_chunk - len;
        }
      }
      n_entries += len;
      uint32_t v = t, dv = len ? d : 0u, written = 0;   // no backtrack when t is unreachable or adjacent
      uint32_t vb = tb, ve = te;                        // v's in-row
      // W of the next step when known without a summing pass: the raw count
      // of v, i.e. the sum of its predecessors' counts (a ring sum or stored
      // pair count after a shortcut step; sigma'_v itself when v was claimed
      // at a level whose counts were not shifted)
      uint64_t w_next = 0;
      bool ok = true;
      auto stage = [&]() {   // v is the next node of the hyperedge
        if (tid == 0 && hbase + written < a.stage_cap) a.stage[hbase + written] = g.orig_of ? g.orig_of[v] : v;
        ++written;
        --dv;
      };
      // the chosen entry's node and in-row, from the thread that holds it
      auto leave = [&](uint32_t w, uint64_t weight) {
        sh.pk[1] = w;
        sh.pk_weight = weight;
      };
      uint32_t p0 = 0, p1 = 0;   // rows of a step by recounting
      if (dv && shortcut && rings) {
        // step from t through level d-1: weights ring (the last test's) of
        // t's in-neighbours, in ascending order
        const uint32_t pi = block_pick<BLOCK>(
            dt,
            [&](uint32_t j0, uint32_t cnt, uint64_t* x) {
              for (uint32_t k = 0; k < kPickPer; ++k)
                if (k < cnt) x[k] = sh.ring[j0 + k];
            },
            [&](uint32_t, uint32_t j, uint64_t weight) { leave(g.in_idx[tb + j], weight); }, 0, st, sh, co);
        if (pi == kUnseen) {
          ok = false;
        } else {
          v = uniform_u32(sh.pk[1]);
          w_next = uniform_u64(sh.pk_weight);
          p0 = sh.poff[pi];
          const uint32_t pn = (pi + 1 < dt ? sh.poff[pi + 1] : pairs) - p0;
          vb = sh.rrs[pi] + p0;
          ve = vb + pn;
          stage();
          if (shortcut == 3) p1 = p0 + pn;
        }
      } else if (dv && shortcut) {
        p1 = dt;
        w_next = uniform_u64(sh.ring[0]);
      }
      if (p1) {
        // step through level L+1 to the row's owner: from w (level L+2) to a
        // u of the pairs (w, u), rows [p0, p1), or from a t without the ring
        // cache to one of its in-neighbours.  The weights, the owners' raw
        // counts, are counted again (the tests kept only their sum).
        const uint64_t r = bounded(st, w_next);
        uint64_t run = 0;
        ok = false;
        for (uint32_t cb = p0; cb < p1; cb += BLOCK) {
          uint32_t r0, dg;
          row_of(rings, cb + tid, p1, &r0, &dg);
          const uint64_t raw = raw_counts_chunk<BLOCK>(g.in_idx, vis, r0, dg, sh, co, sp);
          uint64_t tot;
          const uint64_t excl = run + co.scan(raw, &tot);
          if (run + tot > r) {
            if (excl <= r && r < excl + raw) {
              sh.pk[2] = r0;
              sh.pk[3] = r0 + dg;
              leave(rings ? wg_ld_u32(&pu[cb + tid]) : g.in_idx[tb + cb + tid], raw);
            }
            ok = true;
            break;
          }
          run += tot;
        }
        __syncthreads();
        if (ok) {
          v = uniform_u32(sh.pk[1]);
          vb = uniform_u32(sh.pk[2]);
          ve = uniform_u32(sh.pk[3]);
          w_next = uniform_u64(sh.pk_weight);
          stage();
        }
      }
      // steps through produced levels.  The predecessors of v, at level
      // want + 1, are its visited in-neighbours placed before that level's
      // start: a visited in-neighbour is on level want or above.
      uint32_t start = le;   // of v's level (t's own is not produced past L)
      while (ok && dv >= 2) {
        const uint32_t want = dv - 1;
        const uint32_t below = want == L ? lb : last_start(starts, start);
        // a known W spares rows longer than one pick round their summing pass
        const uint64_t wk = ve - vb > uint32_t(BLOCK) * kPickPer ? w_next : 0ull;
        uint32_t w[kPickPer], wb[kPickPer], we[kPickPer];
        const uint32_t j = block_pick<BLOCK>(
            ve - vb,
            [&](uint32_t j0, uint32_t cnt, uint64_t* x) {
              uint32_t p[kPickPer];
#pragma unroll
              for (uint32_t k = 0; k < kPickPer; ++k) w[k] = k < cnt ? g.in_idx[vb + j0 + k] : 0u;
#pragma unroll
              for (uint32_t k = 0; k < kPickPer; ++k) {
                p[k] = kUnseen;
                wb[k] = we[k] = 0;
                if (k < cnt && vis.maybe(w[k])) {   // all three loads in flight together
                  p[k] = vis.place(w[k]);
                  wb[k] = g.in_ptr[w[k]];
                  we[k] = g.in_ptr[w[k] + 1];
                }
              }
#pragma unroll
              for (uint32_t k = 0; k < kPickPer; ++k)
                if (p[k] < start) x[k] = wg_ld_u64(&vis.sig[p[k]]);
            },
            [&](uint32_t k, uint32_t, uint64_t weight) {
#pragma unroll
              for (uint32_t i = 0; i < kPickPer; ++i)
                if (i == k) {
                  sh.pk[2] = wb[i];
                  sh.pk[3] = we[i];
                  leave(w[i], weight);
                }
            },
            wk, st, sh, co);
        if (j == kUnseen) {
          ok = false;
          break;
        }
        v = uniform_u32(sh.pk[1]);
        vb = uniform_u32(sh.pk[2]);
        ve = uniform_u32(sh.pk[3]);
        start = below;
        w_next = want < 64 && !((shifted >> want) & 1ull) ? uniform_u64(sh.pk_weight) : 0ull;
        stage();
      }
      if (tid == 0) {
        if (!ok) atomicOr(a.flags, kErrBacktrack);
        a.stage_pos[out] = hbase;
        a.he_len[out] = len;
        if (a.st_out) {
          a.st_out[2 * size_t(out)] = s0;
          a.st_out[2 * size_t(out) + 1] = t0;
        }
        if (a.dist_out) a.dist_out[out] = d;
      }
    }
    // the map keeps this BFS's stamp (older than any later one); only the
    // dynamic bitmap is cleared.  The barrier ends every use of the item's
    // LDS state.
    __syncthreads();
    const uint32_t nv = BLOCK == kWave ? qn : uniform_u32(sh.qlen);
    n_nodes += nv;
    if (LDS_BITS)
      for (uint32_t i = tid; i < nv; i += BLOCK) dyn_bits[wg_ld_u32(&q[i]) >> 5] = 0;
    if (--in_hand) {
      ++idx;
    } else {
      const uint32_t take = (a.count - idx) / kTakeWhile > gridDim.x ? kTake : 1u;
      if (tid == 0) {
        const uint64_t next = gridDim.x + atomicAdd(reinterpret_cast<unsigned long long*>(a.work),
                                                    static_cast<unsigned long long>(take));
        sh.next = next < a.count ? static_cast<uint32_t>(next) : a.count;
      }
      __syncthreads();
      idx = uniform_u32(sh.next);
      in_hand = take;
    }
    __syncthreads();
  }
  // (a workgroup whose targets all lacked in-neighbours scanned no arc but
  // still gave every source a level)
  if (tid == 0 && a.stats && (n_arcs || n_nodes)) {
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats[0]), static_cast<unsigned long long>(n_arcs));
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats[1]), static_cast<unsigned long long>(n_nodes));
    if (n_entries)
      atomicAdd(reinterpret_cast<unsigned long long*>(a.entries), static_cast<unsigned long long>(n_entries));
  }
}

// Lays the staged hyperedges out in sample order.
__global__ void k_stage_gather(uint32_t count, const uint64_t* stage_pos, const uint32_t* he_len,
                               const uint64_t* rel_off, uint64_t base, const uint32_t* stage, uint64_t* he_off,
                               uint32_t* he_nodes) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i > count) return;
  const uint64_t o = rel_off[i];
  if (he_off) he_off[i] = base + o;
  if (i == count) return;
  if (!he_nodes) return;
  const uint64_t p = stage_pos[i];
  const uint32_t len = he_len[i];
  for (uint32_t x = 0; x < len; ++x) he_nodes[o + x] = stage[p + x];
}

// Launch wrappers for the host side of the sampler (sample_launch.hip).
hipError_t sample_kernel_occupancy(int block, bool lds_bits, bool multi, size_t dyn_lds, int* per_cu) {
  if (lds_bits) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_sample_paths<kLdsBlock, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(dyn_lds));
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k_sample_paths<kLdsBlock, true>, kLdsBlock,
                                                        dyn_lds);
  }
#define CENTRA_OCC(B, M) hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, k_sample_paths<B, false, M>, B, 0)
  switch (block) {
    case 512: return multi ? CENTRA_OCC(512, true) : CENTRA_OCC(512, false);
    case 256: return multi ? CENTRA_OCC(256, true) : CENTRA_OCC(256, false);
    case 64: return multi ? CENTRA_OCC(64, true) : CENTRA_OCC(64, false);
    default: return multi ? CENTRA_OCC(128, true) : CENTRA_OCC(128, false);
  }
#undef CENTRA_OCC
}

size_t sample_lds_variant_bytes() { return sizeof(SampleShared<kLdsBlock>); }

void sample_kernel_launch(const SampleArgs& a, int block, bool lds_bits, bool multi, uint32_t grid, size_t dyn_lds,
                          hipStream_t s) {
  if (lds_bits) {
    hipLaunchKernelGGL((k_sample_paths<kLdsBlock, true>), dim3(grid), dim3(kLdsBlock), dyn_lds, s, a);
    return;
  }
#define CENTRA_LAUNCH(B, M) hipLaunchKernelGGL((k_sample_paths<B, false, M>), dim3(grid), dim3(B), 0, s, a)
  switch (block) {
    case 512:
      if (multi)
        CENTRA_LAUNCH(512, true);
      else
        CENTRA_LAUNCH(512, false);
      break;
    case 256:
      if (multi)
        CENTRA_LAUNCH(256, true);
      else
        CENTRA_LAUNCH(256, false);
      break;
    case 64:
      if (multi)
        CENTRA_LAUNCH(64, true);
      else
        CENTRA_LAUNCH(64, false);
      break;
    default:
      if (multi)
        CENTRA_LAUNCH(128, true);
      else
        CENTRA_LAUNCH(128, false);
      break;
  }
#undef CENTRA_LAUNCH
}

// ---------------------------------------------------------------------------
// Device-wide BFS of a deferred sample.  A few samples of skewed graphs
// flood millions of nodes (R-MAT scale 22: one in about 300k floods the 2M
// nodes its source reaches, 63M arcs), which takes one 128-thread workgroup
// about a second and holds its launch that long.  Such a sample is redrawn
// here with each level expanded by the whole GPU: full levels (no ring
// tests), which give the same levels, normalised counts and predecessor
// weights as the shortcuts do, then the same backtrack over the same word
// stream, so the hyperedge is the one the workgroup kernel would stage.
// The launch that deferred the samples has finished: their node records
// {sigma', tag} lie in its slots' count arrays (cleared first), their queues
// in its slots' queues.
constexpr int kWideBlock = 256;
constexpr unsigned kWideGrid = 2048;
// a level is pulled when the unvisited nodes' in-arcs (plus a quarter of n
// for reading every tag) are fewer than kPullRatio times the frontier's
// out-arcs: a push scans them twice and claims with returning atomics
constexpr uint64_t kPullRatio = 8;
constexpr uint32_t kPullLane = 32;   // in-row entries a lane sums by itself in a pull

// Record accessors: word 0 = sigma', word 1 = tag.  With base = stamp << 32
// the tag of a node at level l of the current BFS is base + (kUnseen - l):
// "claimed by this BFS" is tag >= base, "at level <= L" is
// tag >= base + (kUnseen - L).
__device__ __forceinline__ uint64_t* sig_of(uint64_t* rec, uint32_t v) { return rec + 2 * size_t(v); }
__device__ __forceinline__ uint64_t* tag_of(uint64_t* rec, uint32_t v) { return rec + 2 * size_t(v) + 1; }
__device__ __forceinline__ uint64_t level_tag(uint64_t base, uint32_t level) { return base + (kUnseen - level); }

// ctl: [0] queue length, [1] largest raw count of the new level, [2] 1 if
// t is on the new level, [3] out-arcs of the last level (the cost of
// pushing it), [4] t (traversal id), [5] in-arcs of the visited nodes
// (the graph's in-arcs less the cost of pulling), [6] arcs scanned, [7]
// nodes given a level
__global__ void k_wide_start(SampleArgs a, uint32_t idx, uint64_t base, uint64_t* ctl) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  RolledWordStream st(a.seed, a.first + idx, a.instance, 0);
  const uint32_t s0 = static_cast<uint32_t>(bounded(st, a.n));
  const uint32_t tp = static_cast<uint32_t>(bounded(st, a.n - 1));
  const uint32_t t0 = tp + (tp >= s0 ? 1u : 0u);
  const uint32_t s = a.new_of ? a.new_of[s0] : s0;
  const uint32_t t = a.new_of ? a.new_of[t0] : t0;
  st_u64(tag_of(a.rec, s), level_tag(base, 0));
  st_u64(sig_of(a.rec, s), 1);
  st_u32(&a.q[0], s);
  ctl[0] = 1;
  ctl[1] = 0;
  ctl[2] = 0;
  ctl[3] = a.row_ptr[s + 1] - a.row_ptr[s];
  ctl[4] = t;
  ctl[5] = a.in_ptr[s + 1] - a.in_ptr[s];
  ctl[6] = 0;
  ctl[7] = 1;
}

// Level nl - 1 = queue entries [lb, le) expanded by every workgroup, a
// chunk of kWideBlock frontier nodes at a time, the arcs of a chunk shared by
// the workgroups of a column of the grid (a few hubs make a narrow level of
// millions of arcs, which a workgroup per chunk left to a handful: a flood of
// R-MAT scale 20 took 4.7 ms): pass 0 claims the new
// level's nodes (returning atomic max on the tag; the claimer zeroes the
// count and appends the node, one queue atomic per wave), pass 1 adds each
// frontier node's count to its new-level out-neighbours.
template <int PASS>
__global__ __launch_bounds__(kWideBlock) void k_wide_level(SampleArgs a, uint32_t lb, uint32_t le, uint64_t base,
                                                           uint32_t nl, uint64_t* ctl) {
  __shared__ uint32_t off[kWideBlock], rs[kWideBlock], scan[kWideBlock / kWave + 1];
  __shared__ uint64_t sg[kWideBlock];
  const int tid = threadIdx.x, lane = lane_id();
  const uint64_t tag_new = level_tag(base, nl);
  const uint64_t lane_lt = (1ull << lane) - 1ull;
  uint64_t arcs = 0;
  for (uint64_t cb = lb + uint64_t(blockIdx.x) * kWideBlock; cb < le; cb += uint64_t(gridDim.x) * kWideBlock) {
    const uint64_t i = cb + tid;
    uint32_t deg = 0, r0 = 0;
    uint64_t sw = 0;
    if (i < le) {
      const uint32_t w = ld_u32(&a.q[i]);
      r0 = a.row_ptr[w];
      deg = a.row_ptr[w + 1] - r0;
      if (PASS == 1) sw = ld_u64(sig_of(a.rec, w));
    }
    uint32_t total;
    const uint32_t o = block_excl_scan_u32<kWideBlock>(deg, &total, scan);
    off[tid] = o;
    rs[tid] = r0;
    sg[tid] = sw;
    if (blockIdx.y == 0) arcs += total;
    __syncthreads();
    for (uint32_t e0 = blockIdx.y * kWideBlock; e0 < total; e0 += gridDim.y * kWideBlock) {   // uniform trip count
      const uint32_t e = e0 + tid;
      bool claimed = false;
      uint32_t v = 0;
      if (e < total) {
        int lo = 0, hi = kWideBlock - 1;   // the last j with off[j] <= e (it has arcs)
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (off[mid] <= e)
            lo = mid;
          else
            hi = mid - 1;
        }
        v = a.col_idx[rs[lo] + (e - off[lo])];
        if (PASS == 0) {
          // most arcs of a flood reach visited nodes: a plain look at the
          // tag spares them the returning atomic
          if (ld_u64(tag_of(a.rec, v)) < base)
            claimed = atomicMax(reinterpret_cast<unsigned long long*>(tag_of(a.rec, v)),
                                static_cast<unsigned long long>(tag_new)) < base;
          if (claimed) st_u64(sig_of(a.rec, v), 0);
        } else if (ld_u64(tag_of(a.rec, v)) == tag_new) {
          atomicAdd(reinterpret_cast<unsigned long long*>(sig_of(a.rec, v)), static_cast<unsigned long long>(sg[lo]));
        }
      }
      if (PASS == 0) {
        const uint64_t m = __ballot(claimed);
        if (m) {
          const int leader = __ffsll(static_cast<unsigned long long>(m)) - 1;
          uint64_t wb = 0;
          if (lane == leader)
            wb = atomicAdd(reinterpret_cast<unsigned long long*>(&ctl[0]), static_cast<unsigned long long>(__popcll(m)));
          wb = __shfl(wb, leader, kWave);
          if (claimed) st_u32(&a.q[wb + __popcll(m & lane_lt)], v);
        }
      }
    }
    __syncthreads();   // off, rs and sg are reused by the next chunk
  }
  // arcs is uniform over the workgroup (each chunk's total): one add
  if (PASS == 0 && a.stats && tid == 0 && arcs)
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats[0]), static_cast<unsigned long long>(arcs));
}

// Level nl pulled instead of pushed (late levels of a flood, when the
// unvisited nodes' in-arcs are fewer than the frontier's out-arcs): every
// unvisited node sums the counts of its in-neighbours on level nl - 1; a
// positive sum puts it on level nl with that raw count.  Each node is
// written by its own thread only, so no atomics on the records.
__global__ __launch_bounds__(kWideBlock) void k_wide_pull(SampleArgs a, uint64_t base, uint32_t nl, uint64_t* ctl) {
  __shared__ uint64_t red[kWideBlock / kWave];
  const int lane = lane_id();
  const uint64_t tag_new = level_tag(base, nl), tag_prev = level_tag(base, nl - 1);
  const uint64_t lane_lt = (1ull << lane) - 1ull;
  uint64_t arcs = 0;
  const uint64_t n_pad = (uint64_t(a.n) + kWideBlock - 1) / kWideBlock * kWideBlock;   // uniform trip count
  for (uint64_t v0 = uint64_t(blockIdx.x) * kWideBlock; v0 < n_pad; v0 += uint64_t(gridDim.x) * kWideBlock) {
    const uint64_t v = v0 + threadIdx.x;
    uint32_t ib = 0, ie = 0;
    if (v < a.n && ld_u64(tag_of(a.rec, static_cast<uint32_t>(v))) < base) {
      ib = a.in_ptr[v];
      ie = a.in_ptr[v + 1];
    }
    arcs += ie - ib;
    // a row of up to kPullLane entries by its own lane, a longer one by the
    // wave (hub rows would otherwise hold the level: the wide BFSs of a 2.7M
    // sample launch at directed R-MAT scale 22, 302 -> 158 ms)
    uint64_t raw = 0;
    if (ie - ib <= kPullLane)
      for (uint32_t e = ib; e < ie; ++e) {
        const uint32_t w = a.in_idx[e];
        if (ld_u64(tag_of(a.rec, w)) == tag_prev) raw += ld_u64(sig_of(a.rec, w));
      }
    for (uint64_t m = __ballot(ie - ib > kPullLane); m; m &= m - 1) {
      const int l = __ffsll(static_cast<unsigned long long>(m)) - 1;
      const uint32_t hb = lane_u32(ib, l), he = lane_u32(ie, l);
      uint64_t x = 0;
      for (uint32_t e = hb + lane; e < he; e += kWave) {
        const uint32_t w = a.in_idx[e];
        if (ld_u64(tag_of(a.rec, w)) == tag_prev) x += ld_u64(sig_of(a.rec, w));
      }
      x = wave_sum_u64(x);
      if (lane == l) raw = x;
    }
    const bool claimed = raw != 0;
    if (claimed) {
      st_u64(sig_of(a.rec, static_cast<uint32_t>(v)), raw);
      st_u64(tag_of(a.rec, static_cast<uint32_t>(v)), tag_new);
    }
    const uint64_t m = __ballot(claimed);
    if (m) {
      const int leader = __ffsll(static_cast<unsigned long long>(m)) - 1;
      uint64_t wb = 0;
      if (lane == leader)
        wb = atomicAdd(reinterpret_cast<unsigned long long*>(&ctl[0]), static_cast<unsigned long long>(__popcll(m)));
      wb = __shfl(wb, leader, kWave);
      if (claimed) st_u32(&a.q[wb + __popcll(m & lane_lt)], static_cast<uint32_t>(v));
    }
  }
  arcs = block_sum_u64<kWideBlock>(arcs, red);
  if (threadIdx.x == 0 && a.stats && arcs)
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats[0]), static_cast<unsigned long long>(arcs));
}

// The new level [le, ne = ctl[0]): its largest raw count into ctl[1]
// (zeroed by the caller), whether t is on it into ctl[2], its size into
// the node statistics.
__global__ __launch_bounds__(kWideBlock) void k_wide_close(SampleArgs a, uint32_t le, uint64_t base, uint32_t nl,
                                                           uint32_t t, uint64_t* ctl) {
  __shared__ uint64_t red[kWideBlock / kWave];
  const uint32_t ne = static_cast<uint32_t>(ctl[0]);
  uint64_t mx = 0, out_arcs = 0, in_arcs = 0;
  for (uint64_t i = le + uint64_t(blockIdx.x) * kWideBlock + threadIdx.x; i < ne; i += uint64_t(gridDim.x) * kWideBlock) {
    const uint32_t v = ld_u32(&a.q[i]);
    const uint64_t x = ld_u64(sig_of(a.rec, v));
    mx = x > mx ? x : mx;
    out_arcs += a.row_ptr[v + 1] - a.row_ptr[v];
    in_arcs += a.in_ptr[v + 1] - a.in_ptr[v];
  }
  mx = block_max_u64<kWideBlock>(mx, red);
  out_arcs = block_sum_u64<kWideBlock>(out_arcs, red);
  in_arcs = block_sum_u64<kWideBlock>(in_arcs, red);
  if (threadIdx.x == 0) {
    if (mx) atomicMax(reinterpret_cast<unsigned long long*>(&ctl[1]), static_cast<unsigned long long>(mx));
    if (out_arcs) atomicAdd(reinterpret_cast<unsigned long long*>(&ctl[3]), static_cast<unsigned long long>(out_arcs));
    if (in_arcs) atomicAdd(reinterpret_cast<unsigned long long*>(&ctl[5]), static_cast<unsigned long long>(in_arcs));
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl[2] = ld_u64(tag_of(a.rec, t)) == level_tag(base, nl) ? 1u : 0u;
    if (a.stats) atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats[1]), static_cast<unsigned long long>(ne - le));
  }
}

// Normalisation of the new level: sigma' = max(1, raw >> shift).
__global__ void k_wide_shift(SampleArgs a, uint32_t le, uint32_t ne, uint32_t shift) {
  for (uint64_t i = le + uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < ne; i += uint64_t(gridDim.x) * blockDim.x) {
    uint64_t* p = sig_of(a.rec, ld_u32(&a.q[i]));
    const uint64_t x = ld_u64(p) >> shift;
    st_u64(p, x ? x : 1ull);
  }
}

// The backtrack of the sample (t at distance d, kUnseen if unreachable) by
// one workgroup over the same word stream as the workgroup kernel (the
// pair's words, then one bounded draw per step), staged the same way.
__global__ __launch_bounds__(kWideBlock) void k_wide_backtrack(SampleArgs a, uint32_t idx, uint64_t base, uint32_t d) {
  __shared__ SampleShared<kWideBlock> sh;
  Coll<kWideBlock> co{sh.red, 0};
  const int tid = threadIdx.x;
  RolledWordStream st(a.seed, a.first + idx, a.instance, 0);
  const uint32_t s0 = static_cast<uint32_t>(bounded(st, a.n));
  const uint32_t tp = static_cast<uint32_t>(bounded(st, a.n - 1));
  const uint32_t t0 = tp + (tp >= s0 ? 1u : 0u);
  const uint32_t t = a.new_of ? a.new_of[t0] : t0;
  const uint32_t len = (d != kUnseen && d >= 2) ? d - 1 : 0u;
  uint64_t hbase = 0;   // thread 0 only
  if (tid == 0 && len) {
    hbase = atomicAdd(reinterpret_cast<unsigned long long*>(a.stage_used), static_cast<unsigned long long>(len));
    atomicAdd(reinterpret_cast<unsigned long long*>(a.entries), static_cast<unsigned long long>(len));
  }
  uint32_t v = t, dv = len ? d : 0u, written = 0;
  bool ok = true;
  while (dv >= 2) {
    const uint32_t want = dv - 1;
    const uint64_t tag_want = level_tag(base, want);
    const uint32_t vb = a.in_ptr[v], ve = a.in_ptr[v + 1];
    const uint32_t j = block_pick<kWideBlock>(
        ve - vb,
        [&](uint32_t j0, uint32_t cnt, uint64_t* x) {
          for (uint32_t k = 0; k < kPickPer; ++k) {
            if (k >= cnt) continue;
            const uint32_t w = a.in_idx[vb + j0 + k];
            const uint64_t tg = ld_u64(tag_of(a.rec, w));
            const uint64_t c = ld_u64(sig_of(a.rec, w));
            x[k] = tg == tag_want ? c : 0ull;
          }
        },
        [](uint32_t, uint32_t, uint64_t) {}, 0, st, sh, co);
    if (j == kUnseen) {
      ok = false;
      break;
    }
    v = a.in_idx[vb + j];
    if (tid == 0 && hbase + written < a.stage_cap) a.stage[hbase + written] = caller_id(a, v);
    ++written;
    --dv;
  }
  if (tid == 0) {
    if (!ok) atomicOr(a.flags, kErrBacktrack);
    a.stage_pos[idx] = hbase;
    a.he_len[idx] = len;
    if (a.st_out) {
      a.st_out[2 * size_t(idx)] = s0;
      a.st_out[2 * size_t(idx) + 1] = t0;
    }
    if (a.dist_out) a.dist_out[idx] = d;
  }
}

int wide_samples(const SampleArgs& a_in, const uint32_t* idx, uint32_t n_items, uint64_t* ctl, uint64_t* host_ctl,
                 uint64_t* arcs, hipStream_t s) {
  // per sample j: records j of a_in.rec (cleared here), slot j's queue, ctl + 8 j
  fill_u64(a_in.rec, 0, size_t(n_items) * 2 * a_in.slot_stride, s);
  struct Walk {
    SampleArgs a;
    uint64_t base, push_cost, visited_in;
    uint32_t t, lb, le, L, d;
    bool live;
  };
  std::vector<Walk> w(n_items);
  for (uint32_t j = 0; j < n_items; ++j) {
    Walk& x = w[j];
    x.a = a_in;
    x.a.rec = a_in.rec + 2 * size_t(j) * a_in.slot_stride;
    x.a.q = a_in.q + size_t(j) * a_in.slot_stride;
    x.a.stats = ctl + 8 * size_t(j) + 6;   // its arcs and nodes, apart from the workgroup kernel's
    x.base = uint64_t(1) << 32;
    hipLaunchKernelGGL(k_wide_start, dim3(1), dim3(64), 0, s, x.a, idx[j], x.base, ctl + 8 * size_t(j));
  }
  const size_t ctl_bytes = size_t(n_items) * 8 * 8;
  if (hipMemcpyAsync(host_ctl, ctl, ctl_bytes, hipMemcpyDeviceToHost, s) != hipSuccess) return CENTRA_EHIP;
  if (hipStreamSynchronize(s) != hipSuccess) return CENTRA_EHIP;
  for (uint32_t j = 0; j < n_items; ++j) {
    Walk& x = w[j];
    x.t = static_cast<uint32_t>(host_ctl[8 * j + 4]);
    x.lb = 0;
    x.le = 1;
    x.L = 0;
    x.d = kUnseen;
    x.live = true;
    x.push_cost = host_ctl[8 * j + 3];
    x.visited_in = host_ctl[8 * j + 5];
  }
  // rounds: every live sample expands one level (pushed, or pulled when the
  // unvisited nodes' in-arcs cost less than pushing the frontier twice)
  // and closes it; one synchronisation per round reads every sample's new
  // level size, maximum, costs and whether t is on it
  for (uint32_t live = n_items; live;) {
    for (uint32_t j = 0; j < n_items; ++j) {
      Walk& x = w[j];
      if (!x.live) continue;
      uint64_t* c = ctl + 8 * size_t(j);
      const uint32_t nl = x.L + 1;
      const uint64_t pull_cost = (x.a.n_arcs - x.visited_in) + x.a.n / 4;
      fill_u64(c + 1, 0, 3, s);
      if (pull_cost < kPullRatio * x.push_cost) {
        hipLaunchKernelGGL(k_wide_pull, dim3(kWideGrid), dim3(kWideBlock), 0, s, x.a, x.base, nl, c);
      } else {
        const unsigned chunks = std::min<uint64_t>(kWideGrid, (uint64_t(x.le - x.lb) + kWideBlock - 1) / kWideBlock);
        // as many workgroups per chunk as the level's arcs keep busy
        const uint64_t rounds = x.push_cost / (uint64_t(chunks) * kWideBlock) + 1;
        const unsigned share = std::min<uint64_t>(std::max(1u, kWideGrid / chunks), rounds);
        const dim3 grid(chunks, share);
        hipLaunchKernelGGL(k_wide_level<0>, grid, dim3(kWideBlock), 0, s, x.a, x.lb, x.le, x.base, nl, c);
        hipLaunchKernelGGL(k_wide_level<1>, grid, dim3(kWideBlock), 0, s, x.a, x.lb, x.le, x.base, nl, c);
      }
      hipLaunchKernelGGL(k_wide_close, dim3(kWideGrid), dim3(kWideBlock), 0, s, x.a, x.le, x.base, nl, x.t, c);
    }
    if (hipMemcpyAsync(host_ctl, ctl, ctl_bytes, hipMemcpyDeviceToHost, s) != hipSuccess) return CENTRA_EHIP;
    if (hipStreamSynchronize(s) != hipSuccess) return CENTRA_EHIP;
    for (uint32_t j = 0; j < n_items; ++j) {
      Walk& x = w[j];
      if (!x.live) continue;
      const uint64_t* h = host_ctl + 8 * size_t(j);
      const uint32_t nl = x.L + 1, ne = static_cast<uint32_t>(h[0]);
      if (ne == x.le || h[2]) {   // nothing new (t unreachable), or t on level nl
        x.d = ne == x.le ? kUnseen : nl;
        x.live = false;
        --live;
        continue;
      }
      uint32_t bl = 0;
      for (uint64_t v = h[1]; v; v >>= 1) ++bl;
      const uint32_t shift = bl > x.a.c_bits ? bl - x.a.c_bits : 0u;
      if (shift) {
        const unsigned gc = std::min<uint64_t>(kWideGrid, (uint64_t(ne - x.le) + kWideBlock - 1) / kWideBlock);
        hipLaunchKernelGGL(k_wide_shift, dim3(gc), dim3(kWideBlock), 0, s, x.a, x.le, ne, shift);
      }
      x.push_cost = h[3];
      x.visited_in = h[5];
      x.lb = x.le;
      x.le = ne;
      x.L = nl;
    }
  }
  for (uint32_t j = 0; j < n_items; ++j)
    hipLaunchKernelGGL(k_wide_backtrack, dim3(1), dim3(kWideBlock), 0, s, w[j].a, idx[j], w[j].base, w[j].d);
  if (hipGetLastError() != hipSuccess) return CENTRA_EHIP;
  if (hipMemcpyAsync(host_ctl, ctl, ctl_bytes, hipMemcpyDeviceToHost, s) != hipSuccess) return CENTRA_EHIP;
  if (hipStreamSynchronize(s) != hipSuccess) return CENTRA_EHIP;
  *arcs = 0;
  for (uint32_t j = 0; j < n_items; ++j) *arcs += host_ctl[8 * j + 6];
  return CENTRA_OK;
}

void stage_gather_launch(uint32_t count, const uint64_t* stage_pos, const uint32_t* he_len, const uint64_t* rel_off,
                         uint64_t base, const uint32_t* stage, uint64_t* he_off, uint32_t* he_nodes, hipStream_t s) {
  hipLaunchKernelGGL(k_stage_gather, dim3((count + 1 + 255) / 256), dim3(256), 0, s, count, stage_pos, he_len, rel_off,
                     base, stage, he_off, he_nodes);
}

}  // namespace centra
