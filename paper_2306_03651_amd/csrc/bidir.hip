// The balanced bidirectional path sampler on gfx950 (the sampling procedure
// of Sec. 5): for sample x, a uniform pair s != t from the Philox stream
// (seed, x, instance, tag 7), a search from s over out-arcs and one from t
// over in-arcs, level by level with normalised counts (forward budget from
// the largest in-degree, backward budget from the largest out-degree; a
// level whose largest raw count needs more bits is shifted right and
// clamped to >= 1).  Each step expands the side whose last level has fewer
// arcs to scan (the forward side on ties).  The first new level that meets
// the other side's last level gives d(s,t) = a + b and the meeting set M
// (every shortest path crosses M once).  One node of M is drawn, in
// ascending caller id, with weight sigma_f * sigma_b (the 128-bit product
// shifted so that the weights of M sum below 2^63, clamped to >= 1); the
// path is then walked from it to t over the backward counts (successors in
// row order) and to s over the forward counts (predecessors in row order),
// one draw per step above level 1.  The hyperedge is the path's internal
// nodes, t's neighbour first; it is empty, with no draw after the pair,
// when t is unreachable or adjacent to s.
//
// One workgroup runs one search at a time over a persistent grid, taking
// work items from an atomic counter.  Each side keeps, per slot, records
// {sigma' u64, tag u64} (tag = stamp << 32 | (kUnseen - level), as in the
// single-source sampler, so nothing is reset between samples) and a queue
// of its nodes in level order.  Only its own workgroup touches a slot, so no
// record is updated atomically: a round takes kPer arcs per thread, sums the
// counts of arcs with the same target in an LDS table, and the thread that
// entered a target there reads, changes and writes its record.  The same
// thread appends a new node, adds its row to the level's cost and checks it
// against the other side's last level, so a level takes one pass over its
// arcs and none over its nodes (unless its counts may need the shift).  A
// record is read only if the node's bit in the side's LDS filter is set.
//
// The level that meets the other side is most of a search, and of its nodes
// only the meeting set's matter.  So each level's arcs are first only read:
// targets whose bit is set in the other side's filter are checked against
// that side's last level, and the counts of those on it are summed in the
// table.  If there are any, and no shift can be due, the search is over
// without a record or queue entry of that level (or only those of the meeting
// set, if the table cannot hold it); if there are none, the level is expanded.  Integer sums and maxima make every count, and so every hyperedge,
// independent of thread timing.
//
// What bounds a search is its chain of dependent trips to memory, three or
// four per round, so the device is filled with as many searches as it holds
// rather than with threads per search.  (With the claims and sums as global
// atomics, which execute in memory on this card, in two passes, and a search
// for the meeting node over the whole last level: BA n = 10^5, 100,000
// samples, 1,600 arcs each, 33.2 ms with 256 threads; with 64, records read
// for every arc and the last level expanded, 10.4 ms, 6 TB/s of records; now
// 2.6 ms.)
#include <stdlib.h>
#include <string.h>

#include "common.hpp"
#include "internal.hpp"

namespace centra {

namespace {

struct BiArgs {
  uint32_t n, c_f, c_b;
  const uint32_t* row_ptr;
  const uint32_t* col_idx;
  const uint32_t* in_ptr;
  const uint32_t* in_idx;
  const uint32_t* new_of;
  const uint32_t* orig_of;
  uint64_t seed;
  uint32_t instance;
  uint64_t first;
  uint32_t count;
  uint32_t stamp0;
  uint64_t slot_stride;
  uint64_t* rec_f;   // slots * stride records {sigma, tag}
  uint64_t* rec_b;
  uint32_t* q_f;     // slots * stride
  uint32_t* q_b;
  uint32_t* work;    // next item (from gridDim.x)
  uint32_t* stage;
  uint64_t stage_cap;
  uint64_t* stage_used;
  uint64_t* stage_pos;
  uint32_t* he_len;
  uint32_t* st_out;
  uint32_t* dist_out;
  uint32_t* flags;
  uint64_t* stats;   // [0] arcs scanned, [1] nodes given a level
};

__device__ __forceinline__ uint64_t* bsig(uint64_t* rec, uint32_t v) { return rec + 2 * size_t(v); }
__device__ __forceinline__ uint64_t* btag(uint64_t* rec, uint32_t v) { return rec + 2 * size_t(v) + 1; }
__device__ __forceinline__ uint64_t blevel_tag(uint64_t base, uint32_t level) { return base + (kUnseen - level); }

__device__ __forceinline__ uint32_t bi_caller(const BiArgs& a, uint32_t v) { return a.orig_of ? a.orig_of[v] : v; }

constexpr int kPer = 2;   // arcs a thread takes per round

template <int BLOCK>
struct BiShared {
  static constexpr uint32_t kTab = 2 * kPer * BLOCK;   // half full at most in a round
  static constexpr uint32_t kMeet = 3 * BLOCK;         // meeting nodes kept in LDS
  static constexpr uint32_t kFilter = 8 * BLOCK;       // words of a side's filter: 16,384 bits for one wave
  uint64_t sum[kTab];   // 0 between rounds
  uint64_t sg[BLOCK];
  uint64_t red[2 * Coll<BLOCK>::kHalf];
  uint32_t key[kTab];   // kUnseen between rounds
  uint32_t off[BLOCK];
  uint32_t rs[BLOCK];
  uint32_t m_id[kMeet];
  uint32_t filter[2][kFilter];
  uint64_t c_sg[2][BLOCK];   // a side's last level, if it is cached: counts, rows, degrees
  uint32_t c_rs[2][BLOCK], c_deg[2][BLOCK];
  uint32_t next, tail, meet, full;
};

// One side of a search: its rows, records, queue, last level q[lo, hi) at
// distance level, the arcs that level would scan and the count budget.
struct Side {
  const uint32_t* ptr;
  const uint32_t* idx;
  uint64_t* rec;
  uint32_t* q;
  uint32_t lo, hi, level, c_bits;
  uint32_t* filter;   // bit v mod its size is set for every node v with a level
  uint64_t cost;
  uint32_t at;        // its place in the caches
  bool cached;
};

template <int BLOCK>
__device__ __forceinline__ bool in_filter(const uint32_t* filter, uint32_t v) {
  return filter[(v >> 5) & (BiShared<BLOCK>::kFilter - 1)] >> (v & 31u) & 1u;
}
template <int BLOCK>
__device__ __forceinline__ void to_filter(uint32_t* filter, uint32_t v) {
  atomicOr(&filter[(v >> 5) & (BiShared<BLOCK>::kFilter - 1)], 1u << (v & 31u));
}

template <int BLOCK>
__device__ __forceinline__ void clear_table(BiShared<BLOCK>& sh) {
  for (uint32_t i = threadIdx.x; i < BiShared<BLOCK>::kTab; i += BLOCK) {
    sh.key[i] = kUnseen;
    sh.sum[i] = 0;
  }
}

// Adds w to the table's sum for v; returns v's slot (kUnseen: none of its
// `probes` first places is free), *won if v was not in the table.
template <int BLOCK>
__device__ __forceinline__ uint32_t to_table(BiShared<BLOCK>& sh, uint32_t v, uint64_t w, bool* won,
                                             uint32_t probes = BiShared<BLOCK>::kTab) {
  constexpr uint32_t kTab = BiShared<BLOCK>::kTab;
  const uint32_t h = (v * 0x9E3779B1u) >> 16;
  *won = false;
  for (uint32_t p = 0; p < probes; ++p) {
    const uint32_t slot = (h + p) & (kTab - 1);
    const uint32_t old = atomicCAS(&sh.key[slot], kUnseen, v);
    if (old != kUnseen && old != v) continue;
    *won = old == kUnseen;
    atomicAdd(reinterpret_cast<unsigned long long*>(&sh.sum[slot]), static_cast<unsigned long long>(w));
    return slot;
  }
  return kUnseen;
}

// The rows of a chunk of x's last level, from place c, in sh; returns their
// arcs.  (A cached level is one chunk.)
template <int BLOCK>
__device__ __forceinline__ uint32_t load_chunk(const Side& x, uint32_t c, BiShared<BLOCK>& sh, Coll<BLOCK>& co) {
  const uint32_t tid = threadIdx.x;
  uint32_t deg = 0, rs = 0;
  uint64_t sg = 0;
  if (x.cached) {
    if (c + tid < x.hi) {
      rs = sh.c_rs[x.at][tid];
      deg = sh.c_deg[x.at][tid];
      sg = sh.c_sg[x.at][tid];
    }
  } else if (c + tid < x.hi) {
    const uint32_t u = wg_ld_u32(&x.q[c + tid]);
    rs = x.ptr[u];
    deg = x.ptr[u + 1] - rs;
    sg = wg_ld_u64(bsig(x.rec, u));
  }
  uint64_t total;
  sh.off[tid] = static_cast<uint32_t>(co.scan(deg, &total));
  sh.rs[tid] = rs;
  sh.sg[tid] = sg;
  __syncthreads();
  return static_cast<uint32_t>(total);   // (below n_arcs < 2^32)
}

// Arcs e0 + k * BLOCK + tid of the chunk's `total`: target (kUnseen past the
// end) and its source's count.
template <int BLOCK, int PER>
__device__ __forceinline__ void load_arcs(const Side& x, uint32_t e0, uint32_t total, const BiShared<BLOCK>& sh,
                                          uint32_t (&v)[PER], uint64_t (&w)[PER]) {
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const uint32_t e = e0 + k * BLOCK + threadIdx.x;
    // the source: the last j with off[j] <= e (sources without arcs repeat
    // the next offset)
    uint32_t l = 0;
#pragma unroll
    for (uint32_t step = BLOCK / 2; step; step >>= 1)
      if (sh.off[l + step] <= e) l += step;
    w[k] = sh.sg[l];
    v[k] = e < total ? x.idx[sh.rs[l] + (e - sh.off[l])] : kUnseen;
  }
}

// Expands x's last level of at most BLOCK nodes and kMeet arcs (otherwise as
// expand_level): the new level is put together in the table, so that its
// counts are final, and normalised, before anything is written, and is cached
// for its own expansion if it is that small again.  Narrow levels are chains
// of trips to memory, here two (targets, their rows) where expand_level takes
// eight.  (4-neighbour grid 64 x 64, 20,000 samples, 43 levels each: 16.4 ms as it
// was, 5.4 now.)
template <int BLOCK>
__device__ __forceinline__ void expand_small(Side& x, const Side& y, uint64_t base, bool exact, BiShared<BLOCK>& sh,
                                             Coll<BLOCK>& co, uint64_t& n_arcs) {
  using S = BiShared<BLOCK>;
  constexpr int PER = S::kMeet / BLOCK, OWN = S::kTab / BLOCK;
  const uint32_t tid = threadIdx.x;
  const uint64_t newtag = blevel_tag(base, x.level + 1), meet_tag = blevel_tag(base, y.level);
  const uint32_t total = load_chunk(x, x.lo, sh, co);
  n_arcs += total;
  uint32_t v[PER];
  uint64_t w[PER];
  load_arcs(x, 0, total, sh, v, w);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    // (a node of this level enters the filter below: a set bit means an
    // earlier level, or another node's bit where the filter is not exact)
    if (v[k] == kUnseen || (in_filter<BLOCK>(x.filter, v[k]) && (exact || wg_ld_u64(btag(x.rec, v[k])) >= base)))
      continue;
    bool won;
    (void)to_table(sh, v[k], w[k], &won);   // (a quarter of the table is free)
  }
  __syncthreads();
  uint32_t u[OWN], cnt = 0;
  uint64_t sg[OWN], mx = 0;
#pragma unroll
  for (int j = 0; j < OWN; ++j) {
    const uint32_t i = j * BLOCK + tid;
    u[j] = sh.key[i];
    sg[j] = sh.sum[i];
    sh.key[i] = kUnseen;
    sh.sum[i] = 0;
    cnt += u[j] != kUnseen ? 1u : 0u;
    mx = sg[j] > mx ? sg[j] : mx;
  }
  uint64_t size;
  uint32_t at = x.hi + static_cast<uint32_t>(co.scan(cnt, &size));
  const uint32_t bl = bitlen64(co.max(mx));
  const uint32_t shift = bl > x.c_bits ? bl - x.c_bits : 0u;
  uint64_t cost = 0;
  const bool cache = size <= BLOCK;
#pragma unroll
  for (int j = 0; j < OWN; ++j) {
    if (u[j] == kUnseen) continue;
    const uint64_t c = sg[j] >> shift ? sg[j] >> shift : 1ull;
    wg_st_u64(bsig(x.rec, u[j]), c);
    wg_st_u64(btag(x.rec, u[j]), newtag);
    wg_st_u32(&x.q[at], u[j]);
    to_filter<BLOCK>(x.filter, u[j]);
    const uint32_t rs = x.ptr[u[j]], deg = x.ptr[u[j] + 1] - rs;
    cost += deg;
    if (cache) {
      sh.c_rs[x.at][at - x.hi] = rs;
      sh.c_deg[x.at][at - x.hi] = deg;
      sh.c_sg[x.at][at - x.hi] = c;
    }
    if (in_filter<BLOCK>(y.filter, u[j]) && wg_ld_u64(btag(y.rec, u[j])) == meet_tag) {
      const uint32_t i = atomicAdd(&sh.meet, 1u);
      if (i < S::kMeet) sh.m_id[i] = u[j];
    }
    ++at;
  }
  x.lo = x.hi;
  x.hi += static_cast<uint32_t>(size);
  ++x.level;
  x.cached = cache;
  x.cost = co.sum(cost);   // (a barrier: records, caches and sh.meet are as the next level finds them)
  __syncthreads();
}

// Looks for the next level of x on y's last level.  kMet: it meets, and the
// table holds the meeting set with its counts (sh.meet nodes).  Otherwise the
// table is as between rounds and the level is to be expanded: kMetMany: it
// meets in more nodes than the table holds, which alone matter; kUnmet: it
// does not meet, or a shift may be due.
enum Ahead { kUnmet, kMet, kMetMany };
template <int BLOCK>
__device__ __forceinline__ Ahead look_ahead(const Side& x, const Side& y, uint64_t base, BiShared<BLOCK>& sh,
                                           Coll<BLOCK>& co, uint64_t* arcs) {
  using S = BiShared<BLOCK>;
  constexpr int PER = 4;
  const uint32_t tid = threadIdx.x;
  const uint64_t meet_tag = blevel_tag(base, y.level);
  uint64_t weight = 0;   // saturating
  *arcs = 0;
  for (uint32_t c = x.lo; c < x.hi; c += BLOCK) {
    const uint32_t total = load_chunk(x, c, sh, co);
    *arcs += total;
    for (uint32_t e0 = 0; e0 < total; e0 += PER * BLOCK) {
      uint32_t v[PER];
      uint64_t w[PER];
      load_arcs(x, e0, total, sh, v, w);
      const bool full = *const_cast<const volatile uint32_t*>(&sh.full) != 0;   // (once set, the table is of no use)
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        if (v[k] == kUnseen) continue;
        weight = sat_add(weight, w[k]);
        if (full || !in_filter<BLOCK>(y.filter, v[k]) || wg_ld_u64(btag(y.rec, v[k])) != meet_tag) continue;
        bool won;
        const uint32_t slot = to_table(sh, v[k], w[k], &won, 32u);
        if (won && atomicAdd(&sh.meet, 1u) >= S::kMeet) sh.full = 1;
        if (slot == kUnseen) sh.full = 1;
      }
    }
    __syncthreads();   // the chunk is read
  }
  const bool fits = bitlen64(co.sat_sum(weight)) <= x.c_bits;
  const bool met = uniform_u32(sh.meet) != 0;
  const bool full = uniform_u32(sh.full) != 0;
  if (met && fits && !full) return kMet;
  if (met) {
    __syncthreads();
    clear_table(sh);
    if (tid == 0) {
      sh.meet = 0;
      sh.full = 0;
    }
    __syncthreads();
  }
  return met && fits ? kMetMany : kUnmet;
}

// Expands x's last level: the next level is appended to its queue, its counts
// normalised (only: just its nodes on y's last level); sh.meet counts its nodes
// on y's last level, the first kMeet of them in sh.m_id.  Uniform control flow; contains barriers.
template <int BLOCK>
__device__ __forceinline__ void expand_level(Side& x, const Side& y, uint64_t base, bool only, BiShared<BLOCK>& sh,
                                             Coll<BLOCK>& co) {
  using S = BiShared<BLOCK>;
  const uint32_t tid = threadIdx.x;
  const uint64_t newtag = blevel_tag(base, x.level + 1), meet_tag = blevel_tag(base, y.level);
  uint64_t cost = 0, weight = 0;   // of the thread's new nodes, of its arcs into the new level (saturating)
  for (uint32_t c = x.lo; c < x.hi; c += BLOCK) {
    const uint32_t total = load_chunk(x, c, sh, co);
    uint32_t v[kPer];
    uint64_t w[kPer];
    load_arcs(x, 0, total, sh, v, w);
    for (uint32_t e0 = 0; e0 < total; e0 += kPer * BLOCK) {
      uint32_t u[kPer], slot[kPer];
      uint64_t tag[kPer], sig[kPer], wk[kPer];
      bool won[kPer];
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        u[k] = v[k];
        wk[k] = w[k];
        if (only && u[k] != kUnseen &&
            !(in_filter<BLOCK>(y.filter, u[k]) && wg_ld_u64(btag(y.rec, u[k])) == meet_tag))
          u[k] = kUnseen;
        const bool known = u[k] != kUnseen && in_filter<BLOCK>(x.filter, u[k]);
        tag[k] = known ? wg_ld_u64(btag(x.rec, u[k])) : 0ull;
        sig[k] = known ? wg_ld_u64(bsig(x.rec, u[k])) : 0ull;
      }
      if (e0 + kPer * BLOCK < total) load_arcs(x, e0 + kPer * BLOCK, total, sh, v, w);   // the next round's
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        won[k] = false;
        slot[k] = 0;
        if (u[k] == kUnseen || (tag[k] >= base && tag[k] != newtag)) continue;   // none, or on an earlier level
        weight = sat_add(weight, wk[k]);
        slot[k] = to_table(sh, u[k], wk[k], &won[k]);   // (half of the table is free)
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const bool fresh = won[k] && tag[k] != newtag;
        if (won[k]) {
          const uint64_t sum = sh.sum[slot[k]];
          sh.sum[slot[k]] = 0;
          sh.key[slot[k]] = kUnseen;
          wg_st_u64(bsig(x.rec, u[k]), fresh ? sum : sig[k] + sum);
          if (fresh) wg_st_u64(btag(x.rec, u[k]), newtag);
        }
        const uint64_t m = __ballot(fresh);
        if (m) {
          uint32_t at = 0;
          if (lane_id() == 0) at = atomicAdd(&sh.tail, static_cast<uint32_t>(__popcll(m)));
          at = uniform_u32(at) + __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                          __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0));
          if (fresh) {
            wg_st_u32(&x.q[at], u[k]);
            to_filter<BLOCK>(x.filter, u[k]);
            cost += x.ptr[u[k] + 1] - x.ptr[u[k]];
            if (in_filter<BLOCK>(y.filter, u[k]) && wg_ld_u64(btag(y.rec, u[k])) == meet_tag) {
              const uint32_t i = atomicAdd(&sh.meet, 1u);
              if (i < S::kMeet) sh.m_id[i] = u[k];
            }
          }
        }
      }
      __syncthreads();   // records and table are as the next round finds them
    }
  }
  x.cached = false;
  x.lo = x.hi;
  x.hi = uniform_u32(sh.tail);
  ++x.level;
  x.cost = co.sum(cost);
  // normalisation, unless all the level's arcs together stay within the budget
  if (bitlen64(co.sat_sum(weight)) <= x.c_bits) return;
  uint64_t mx = 0;
  for (uint32_t i = x.lo + tid; i < x.hi; i += BLOCK) {
    const uint64_t sg = wg_ld_u64(bsig(x.rec, wg_ld_u32(&x.q[i])));
    mx = sg > mx ? sg : mx;
  }
  const uint32_t bl = bitlen64(co.max(mx));
  const uint32_t shift = bl > x.c_bits ? bl - x.c_bits : 0u;
  if (shift) {
    for (uint32_t i = x.lo + tid; i < x.hi; i += BLOCK) {
      uint64_t* p = bsig(x.rec, wg_ld_u32(&x.q[i]));
      const uint64_t sg = wg_ld_u64(p) >> shift;
      wg_st_u64(p, sg ? sg : 1ull);
    }
    __syncthreads();
  }
}

// 128-bit product's bit length, and the scaled weight.
__device__ __forceinline__ uint32_t bitlen128(unsigned __int128 x) {
  const uint64_t hi = static_cast<uint64_t>(x >> 64);
  return hi ? 64u + bitlen64(hi) : bitlen64(static_cast<uint64_t>(x));
}

// The weight of row entry u (0 if u is not on level `want` of the side
// whose records are rec): its count.
__device__ __forceinline__ uint64_t step_weight(uint64_t* rec, uint32_t u, uint64_t want_tag) {
  const uint64_t tg = wg_ld_u64(btag(rec, u));
  const uint64_t c = wg_ld_u64(bsig(rec, u));
  return tg == want_tag ? c : 0ull;
}

// One walk step: among the entries of row [rb, re) of idx on level `want`
// of the side (records rec), the one drawn with weight sigma (in row
// order).  Draws one word (or more, by rejection).
template <int BLOCK>
__device__ __forceinline__ uint32_t walk_pick(const uint32_t* idx, uint32_t rb, uint32_t re, uint64_t* rec,
                                              uint64_t want_tag, RolledWordStream& st, Coll<BLOCK>& co) {
  // the row's first chunk is kept between the passes
  const uint32_t u0 = rb + threadIdx.x < re ? idx[rb + threadIdx.x] : 0u;
  const uint64_t w0 = rb + threadIdx.x < re ? step_weight(rec, u0, want_tag) : 0ull;
  uint64_t W = w0;
  for (uint32_t c = rb + BLOCK; c < re; c += BLOCK) {
    const uint32_t e = c + threadIdx.x;
    W += e < re ? step_weight(rec, idx[e], want_tag) : 0ull;
  }
  W = co.sum(W);
  if (W == 0) return kUnseen;
  const uint64_t r = bounded(st, W);
  uint64_t run = 0;
  for (uint32_t c = rb; c < re; c += BLOCK) {
    const uint32_t e = c + threadIdx.x;
    const uint32_t u = c == rb ? u0 : e < re ? idx[e] : 0u;
    const uint64_t w = c == rb ? w0 : e < re ? step_weight(rec, u, want_tag) : 0ull;
    uint64_t tot;
    const uint64_t lo = run + co.scan(w, &tot);
    if (run + tot > r) {
      const uint64_t m = co.max(w && lo <= r && r < lo + w ? uint64_t(u) + 1 : 0ull);
      return m ? static_cast<uint32_t>(m - 1) : kUnseen;
    }
    run += tot;
  }
  return kUnseen;
}

// The drawn node of the meeting set, as its caller id: x is the side
// expanded last, y the other; sh.meet nodes.  ahead: the table holds them
// with x's counts; else x's records do, and sh.m_id their first kMeet.
// Their weights are summed in ascending caller id: by a search over the
// caller ids with a pass over LDS each, or, for more nodes than fit there,
// by three or four digits of the ids with a pass over memory each.
template <int BLOCK>
__device__ __forceinline__ uint32_t draw_meeting(const BiArgs& a, const Side& x, const Side& y, uint64_t base,
                                                 bool ahead, RolledWordStream& st, BiShared<BLOCK>& sh,
                                                 Coll<BLOCK>& co) {
  using S = BiShared<BLOCK>;
  const uint32_t tid = threadIdx.x, cnt = uniform_u32(sh.meet);
  const bool few = cnt <= S::kMeet;
  auto product = [&](uint32_t v) {
    return static_cast<unsigned __int128>(wg_ld_u64(bsig(x.rec, v))) * wg_ld_u64(bsig(y.rec, v));
  };
  if (cnt < x.hi - x.lo && !few) {   // the set moves to the front of its level in the queue
    const uint64_t tag = blevel_tag(base, y.level);
    uint32_t done = 0;
    for (uint32_t c = x.lo; c < x.hi; c += BLOCK) {
      const uint32_t v = c + tid < x.hi ? wg_ld_u32(&x.q[c + tid]) : kUnseen;
      const bool in = v != kUnseen && wg_ld_u64(btag(y.rec, v)) == tag;
      uint64_t tot;
      const uint32_t at = static_cast<uint32_t>(co.scan(in ? 1u : 0u, &tot));   // (a barrier: the chunk is read)
      if (in) wg_st_u32(&x.q[x.lo + done + at], v);
      done += static_cast<uint32_t>(tot);
    }
    __syncthreads();
  }
  // the set's places: the table's slots, or 0 .. cnt - 1
  const uint32_t places = ahead ? S::kTab : cnt;
  uint32_t* id = ahead ? sh.key : sh.m_id;   // kUnseen: an empty slot
  uint64_t* weights = sh.sum;                // (of no other use here)
  constexpr uint32_t kOwn = S::kTab / BLOCK;
  static_assert(S::kMeet <= S::kTab, "a place per thread and turn");
  unsigned __int128 own[kOwn];   // the products of the thread's places, if they are few
  uint64_t pb = 0;
  if (few) {
#pragma unroll
    for (uint32_t j = 0; j < kOwn; ++j) {
      const uint32_t i = j * BLOCK + tid;
      const uint32_t v = i < places ? id[i] : kUnseen;
      own[j] = 0;
      if (v == kUnseen) continue;
      own[j] = ahead ? static_cast<unsigned __int128>(sh.sum[i]) * wg_ld_u64(bsig(y.rec, v)) : product(v);
      id[i] = bi_caller(a, v);
      const uint64_t b = bitlen128(own[j]);
      pb = b > pb ? b : pb;
    }
  } else {
    for (uint32_t i = tid; i < cnt; i += BLOCK) {
      const uint64_t b = bitlen128(product(wg_ld_u32(&x.q[x.lo + i])));
      pb = b > pb ? b : pb;
    }
  }
  pb = co.max(pb);
  const uint32_t room = 63u - bitlen64(cnt);
  const uint32_t shift = pb > room ? static_cast<uint32_t>(pb) - room : 0u;
  auto weight = [&](unsigned __int128 p) -> uint64_t {
    const uint64_t w = static_cast<uint64_t>(p >> shift);
    return w ? w : 1ull;
  };
  if (few) {
#pragma unroll
    for (uint32_t j = 0; j < kOwn; ++j)
      if (j * BLOCK + tid < places) weights[j * BLOCK + tid] = own[j] ? weight(own[j]) : 0ull;
    __syncthreads();
    // the sum of the weights of the nodes with caller ids up to `upto`
    auto sum_upto = [&](uint32_t upto) {
      uint64_t sum = 0;
      for (uint32_t i = tid; i < places; i += BLOCK) sum += id[i] <= upto ? weights[i] : 0ull;
      return co.sum(sum);
    };
    const uint64_t r = bounded(st, sum_upto(a.n - 1));
    uint32_t lo = 0, hi = a.n - 1;
    while (lo < hi) {
      const uint32_t mid = lo + (hi - lo) / 2;
      if (sum_upto(mid) > r)
        hi = mid;
      else
        lo = mid + 1;
    }
    return lo;
  }
  // digit by digit from the top, the first pass also giving the total
  constexpr uint32_t kDigit = 8, kOwnBins = (1u << kDigit) > BLOCK ? (1u << kDigit) / BLOCK : 1u;
  static_assert(S::kTab >= (1u << kDigit), "a bin per place");
  uint32_t lo = 0, bits = 32u - static_cast<uint32_t>(__builtin_clz(a.n - 1));
  uint64_t r = 0;
  for (bool first = true; bits; first = false) {
    const uint32_t step = bits < kDigit ? bits : kDigit, rest = bits - step;
    for (uint32_t i = tid; i < 1u << kDigit; i += BLOCK) weights[i] = 0;
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += BLOCK) {
      const uint32_t v = wg_ld_u32(&x.q[x.lo + i]);
      const uint32_t off = bi_caller(a, v) - lo;
      if (bits < 32 && off >> bits) continue;   // (off wraps below lo)
      atomicAdd(reinterpret_cast<unsigned long long*>(&weights[off >> rest]),
                static_cast<unsigned long long>(weight(product(v))));
    }
    __syncthreads();
    uint64_t mine = 0, total;
    for (uint32_t j = 0; j < kOwnBins; ++j)
      if (tid * kOwnBins + j < 1u << kDigit) mine += weights[tid * kOwnBins + j];
    const uint64_t before = co.scan(mine, &total);
    if (first) r = bounded(st, total);
    // the bin that holds r, and r past the bins below it
    if (before <= r && r < before + mine) {
      uint64_t run = before;
      uint32_t d = tid * kOwnBins;
      while (run + weights[d] <= r) run += weights[d++];
      sh.next = d;
      sh.sg[0] = r - run;
    }
    __syncthreads();
    lo += uniform_u32(sh.next) << rest;
    r = uniform_u64(sh.sg[0]);
    bits = rest;
    __syncthreads();
  }
  return lo;
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_sample_bidir(BiArgs a) {
  __shared__ BiShared<BLOCK> sh;
  Coll<BLOCK> co{sh.red, 0};
  const uint32_t tid = threadIdx.x;
  const size_t slot = blockIdx.x;
  uint64_t n_arcs = 0, n_nodes = 0;
  clear_table(sh);
  uint32_t idx = blockIdx.x;
  while (idx < a.count) {
    uint32_t next = 0;
    if (tid == 0) next = atomicAdd(a.work, 1u);   // the next item, under way during this one
    const uint64_t base = uint64_t(a.stamp0 + idx) << 32;
    RolledWordStream st(a.seed, a.first + idx, a.instance, 7);
    const uint32_t s0 = static_cast<uint32_t>(bounded(st, a.n));
    const uint32_t tp = static_cast<uint32_t>(bounded(st, a.n - 1));
    const uint32_t t0 = tp + (tp >= s0 ? 1u : 0u);
    const uint32_t s = a.new_of ? a.new_of[s0] : s0;
    const uint32_t t = a.new_of ? a.new_of[t0] : t0;
    Side x{a.row_ptr, a.col_idx, a.rec_f + 2 * slot * a.slot_stride, a.q_f + slot * a.slot_stride, 0, 1, 0, a.c_f,
           sh.filter[0], a.row_ptr[s + 1] - a.row_ptr[s], 0, false};
    Side y{a.in_ptr, a.in_idx, a.rec_b + 2 * slot * a.slot_stride, a.q_b + slot * a.slot_stride, 0, 1, 0, a.c_b,
           sh.filter[1], a.in_ptr[t + 1] - a.in_ptr[t], 1, false};
    if (tid == 0) {
      wg_st_u64(btag(x.rec, s), blevel_tag(base, 0));
      wg_st_u64(bsig(x.rec, s), 1);
      wg_st_u32(&x.q[0], s);
      wg_st_u64(btag(y.rec, t), blevel_tag(base, 0));
      wg_st_u64(bsig(y.rec, t), 1);
      wg_st_u32(&y.q[0], t);
      sh.meet = 0;
      sh.full = 0;
    }
    for (uint32_t i = tid; i < 2 * BiShared<BLOCK>::kFilter; i += BLOCK) (&sh.filter[0][0])[i] = 0;
    __syncthreads();
    if (tid == 0) {
      to_filter<BLOCK>(x.filter, s);
      to_filter<BLOCK>(y.filter, t);
    }
    uint32_t d = kUnseen;
    bool fwd = true, ahead = false;
    while (x.lo < x.hi && y.lo < y.hi) {
      // x is the side to expand: the forward one on ties
      if (y.cost < x.cost || (y.cost == x.cost && !fwd)) {
        const Side z = x;
        x = y;
        y = z;
        fwd = !fwd;
      }
      if (tid == 0) sh.tail = x.hi;
      __syncthreads();
      if (x.cost <= BiShared<BLOCK>::kMeet && x.hi - x.lo <= BLOCK) {
        expand_small(x, y, base, a.n <= 32 * BiShared<BLOCK>::kFilter, sh, co, n_arcs);
      } else {
        uint64_t arcs;
        const Ahead found = look_ahead(x, y, base, sh, co, &arcs);
        n_arcs += arcs;
        ahead = found == kMet;
        if (ahead)
          ++x.level;
        else
          expand_level(x, y, base, found == kMetMany, sh, co);
      }
      if (uniform_u32(sh.meet)) {
        d = x.level + y.level;
        break;
      }
    }
    n_nodes += x.hi + y.hi;
    const uint32_t f_level = fwd ? x.level : y.level, b_level = d - f_level;
    uint64_t* f_rec = fwd ? x.rec : y.rec;
    uint64_t* b_rec = fwd ? y.rec : x.rec;
    const uint32_t len = (d != kUnseen && d >= 2) ? d - 1 : 0u;
    uint64_t hbase = 0;   // thread 0's
    if (tid == 0 && len)
      hbase = atomicAdd(reinterpret_cast<unsigned long long*>(a.stage_used), static_cast<unsigned long long>(len));
    bool ok = true;
    if (len) {
      const uint32_t m = draw_meeting(a, x, y, base, ahead, st, sh, co);
      auto put = [&](uint32_t at, uint32_t id) {
        if (tid == 0 && hbase + at < a.stage_cap) a.stage[hbase + at] = id;
      };
      if (f_level && b_level) put(b_level - 1, m);   // (else m is s or t)
      const uint32_t vm = a.new_of ? a.new_of[m] : m;
      // first toward t over the backward counts: successors on out-rows, the
      // node at backward level j goes to position j - 1; then toward s over
      // the forward counts: predecessors on in-rows, the node at forward
      // level i goes to position d - 1 - i
      bool back = true;
      uint32_t j = b_level, cur = vm;
      for (;;) {
        if (j < 2) {
          if (!back) break;
          back = false;
          j = f_level;
          cur = vm;
          continue;
        }
        const uint32_t* ptr = back ? a.row_ptr : a.in_ptr;
        cur = walk_pick(back ? a.col_idx : a.in_idx, ptr[cur], ptr[cur + 1], back ? b_rec : f_rec,
                        blevel_tag(base, j - 1), st, co);
        if (cur == kUnseen) {
          ok = false;
          break;
        }
        put(back ? j - 2 : d - j, bi_caller(a, cur));
        --j;
      }
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
      sh.next = next;
    }
    __syncthreads();
    if (d != kUnseen) clear_table(sh);   // the meeting set's places and weights
    idx = uniform_u32(sh.next);
    __syncthreads();
  }
  if (tid == 0 && a.stats && n_arcs) {
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats[0]), static_cast<unsigned long long>(n_arcs));
    atomicAdd(reinterpret_cast<unsigned long long*>(&a.stats[1]), static_cast<unsigned long long>(n_nodes));
  }
}

unsigned grid_cap(uint64_t want, uint32_t cap) { return static_cast<unsigned>(want < cap ? want : cap); }

}  // namespace

constexpr uint32_t kBiManySamples = 16384;
constexpr uint32_t kBiFewSlots = 1024;

// Slot arrays of the bidirectional sampler: forward and backward records
// and queues, 40 bytes per node per slot, at most half of the device's
// memory (the context budget can lower that).
constexpr uint32_t kBiLeanSlots = 1792;   // slots beyond which memory is only taken if much is left
// 32nds of the device for more: a node has twice the state of the path
// sampler's (BA n = 10^6, 100,000 samples: 6.1 ms with 3,584 slots, which take
// 14.8 of them; 6.9 with the 2,900 that 12 hold)
constexpr uint32_t kBiSlotParts = 15;

static size_t most_bidir_slots(centra_ctx* ctx, uint32_t n) {
  const size_t most = slot_mem_cap(ctx) / (size_t(n) * 40);
  return most ? most : 1;
}

static int ensure_bidir_slots(centra_ctx* ctx, uint32_t n, uint32_t want, hipStream_t s) {
  // enough of them, or all that this many were cut down to
  if ((ctx->bi_slots >= want && ctx->bi_n >= n) || (ctx->bi_want >= want && ctx->bi_n == n)) return CENTRA_OK;
  const uint32_t nn = n;   // sized for this launch alone (see ensure_slots)
  DevBuf* bufs[] = {&ctx->bi_rec_f, &ctx->bi_rec_b, &ctx->bi_q_f, &ctx->bi_q_b};
  size_t have = 0;
  for (DevBuf* b : bufs) have += b->bytes;
  uint32_t slots = slots_that_fit(ctx, size_t(nn) * 40, want, kBiLeanSlots, kBiSlotParts, have);
  if (ctx->bi_slots >= slots && ctx->bi_n >= nn) return CENTRA_OK;
  int rc;
  for (;;) {   // halve the slot count while the device cannot hold the state
    for (DevBuf* b : bufs) release(ctx, *b);
    ctx->bi_slots = ctx->bi_want = 0;
    ctx->bi_n = 0;
    rc = ensure(ctx, ctx->bi_rec_f, size_t(slots) * nn * 16, false, s);
    if (!rc) rc = ensure(ctx, ctx->bi_rec_b, size_t(slots) * nn * 16, false, s);
    if (!rc) rc = ensure(ctx, ctx->bi_q_f, size_t(slots) * nn * 4, false, s);
    if (!rc) rc = ensure(ctx, ctx->bi_q_b, size_t(slots) * nn * 4, false, s);
    if (rc != CENTRA_ENOMEM || slots <= 64) break;
    slots /= 2;
  }
  if (rc) return rc;
  fill_u64(static_cast<uint64_t*>(ctx->bi_rec_f.ptr), 0, size_t(slots) * nn * 2, s);   // stamp 0: never claimed
  fill_u64(static_cast<uint64_t*>(ctx->bi_rec_b.ptr), 0, size_t(slots) * nn * 2, s);
  CENTRA_HIP(ctx, hipGetLastError());
  ctx->bi_slots = slots;
  ctx->bi_want = want;
  ctx->bi_n = nn;
  return CENTRA_OK;
}

int sample_bidir_to_stage(centra_ctx* ctx, const centra_graph* g, uint64_t seed, uint32_t instance, uint64_t first,
                          uint32_t count, uint32_t* st_out, uint32_t* dist_out, uint64_t* total, hipStream_t s) {
  int rc;
  *total = 0;
  if (count == 0) return CENTRA_OK;
  // One wave per search where there are searches enough to even out their
  // lengths (BA n = 10^5, 100,000 samples: 2.6 ms, 3.4 with two; 4-neighbour
  // grid 64 x 64: 21 against 32), two below that (directed R-MAT scale 18,
  // 4,000 samples: 1.0 ms with one, 0.62 with two, 0.46 with four; BA n =
  // 10^5: 0.31, 0.24, 0.34; grid, 1,000 samples: 1.3, 1.3, 2.4) and four where
  // memory holds too few slots for more searches to fill the device.
  const char* env = getenv("CENTRA_BIDIR_BLOCK");   // test hook: 64, 128 or 256
  int block = most_bidir_slots(ctx, g->n) < kBiFewSlots ? 256 : count < kBiManySamples ? 128 : 64;
  if (env && (atoi(env) == 64 || atoi(env) == 128 || atoi(env) == 256)) block = atoi(env);
  auto* kernel = block == 64 ? &k_sample_bidir<64> : block == 128 ? &k_sample_bidir<128> : &k_sample_bidir<256>;
  int per_cu = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0) != hipSuccess || per_cu <= 0) per_cu = 1;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device) != hipSuccess || cus <= 0)
    cus = 256;
  (void)hipGetLastError();
  const uint64_t resident = uint64_t(cus) * per_cu;
  if ((rc = ensure_bidir_slots(ctx, g->n, grid_cap(count < resident ? count : resident, 8192), s))) return rc;
  const uint32_t grid = count < ctx->bi_slots ? count : ctx->bi_slots;
  if ((rc = ensure(ctx, ctx->stage_pos, size_t(count) * 8, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->stage_len, size_t(count) * 4 + 8 + 8 * (size_t(count) + 1), false, s))) return rc;
  if ((rc = ensure(ctx, ctx->work_ctr, 64, false, s))) return rc;
  uint64_t cap = size_t(count) * 8 + 1024;
  if (ctx->stage_nodes.bytes / 4 > cap) cap = ctx->stage_nodes.bytes / 4;
  // the count budgets: forward sums run over in-neighbours, backward sums
  // over out-neighbours (a test override lowers both)
  const uint32_t c_f = g->count_bits;
  uint32_t c_b = 63u - (g->max_out_degree ? 32u - static_cast<uint32_t>(__builtin_clz(g->max_out_degree)) : 0u);
  if (g->count_bits_override && g->count_bits_override < c_b) c_b = g->count_bits_override;
  for (int attempt = 0; attempt < 3; ++attempt) {
    if ((rc = ensure(ctx, ctx->stage_nodes, cap * 4, false, s))) return rc;
    cap = ctx->stage_nodes.bytes / 4;
    uint32_t* work = static_cast<uint32_t*>(ctx->work_ctr.ptr);
    uint64_t* used = reinterpret_cast<uint64_t*>(static_cast<char*>(ctx->work_ctr.ptr) + 8);
    fill_u32(work, grid, 1, s);   // (the first items are the workgroups' own)
    fill_u64(used, 0, 1, s);
    if (ctx->stamp_next == 0 || uint64_t(ctx->stamp_next) + count > 0xFFFFFFFFull) {
      // 32-bit stamps would run out: clear every record of both samplers
      fill_u64(static_cast<uint64_t*>(ctx->bi_rec_f.ptr), 0, size_t(ctx->bi_slots) * ctx->bi_n * 2, s);
      fill_u64(static_cast<uint64_t*>(ctx->bi_rec_b.ptr), 0, size_t(ctx->bi_slots) * ctx->bi_n * 2, s);
      if (ctx->slot_map.ptr)
        fill_u64(static_cast<uint64_t*>(ctx->slot_map.ptr), 0, size_t(ctx->slots) * ctx->slot_n, s);
      ctx->stamp_next = 1;
    }
    BiArgs a{};
    a.n = g->n;
    a.c_f = c_f;
    a.c_b = c_b;
    a.row_ptr = g->bfs_row_ptr;
    a.col_idx = g->bfs_col_idx;
    a.in_ptr = g->bfs_in_ptr;
    a.in_idx = g->bfs_in_idx;
    a.new_of = g->new_of;
    a.orig_of = g->orig_of;
    a.seed = seed;
    a.instance = instance;
    a.first = first;
    a.count = count;
    a.stamp0 = ctx->stamp_next;
    ctx->stamp_next += count;
    a.slot_stride = ctx->bi_n;
    a.rec_f = static_cast<uint64_t*>(ctx->bi_rec_f.ptr);
    a.rec_b = static_cast<uint64_t*>(ctx->bi_rec_b.ptr);
    a.q_f = static_cast<uint32_t*>(ctx->bi_q_f.ptr);
    a.q_b = static_cast<uint32_t*>(ctx->bi_q_b.ptr);
    a.work = work;
    a.stage = static_cast<uint32_t*>(ctx->stage_nodes.ptr);
    a.stage_cap = cap;
    a.stage_used = used;
    a.stage_pos = static_cast<uint64_t*>(ctx->stage_pos.ptr);
    a.he_len = static_cast<uint32_t*>(ctx->stage_len.ptr);
    a.st_out = st_out;
    a.dist_out = dist_out;
    a.flags = ctx->d_flags;
    a.stats = reinterpret_cast<uint64_t*>(static_cast<char*>(ctx->work_ctr.ptr) + 16);
    fill_u64(a.stats, 0, 2, s);
    CENTRA_HIP(ctx, hipEventRecord(ctx->ev[6], s));
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), 0, s, a);
    CENTRA_HIP(ctx, hipGetLastError());
    CENTRA_HIP(ctx, hipEventRecord(ctx->ev[7], s));
    uint64_t host_ctr[4] = {0, 0, 0, 0};
    CENTRA_HIP(ctx, hipMemcpyAsync(host_ctr, ctx->work_ctr.ptr, 32, hipMemcpyDeviceToHost, s));
    CENTRA_HIP(ctx, hipStreamSynchronize(s));
    if ((rc = check_flags(ctx, s, "sample_paths_bidir"))) return rc;
    const uint64_t host_used = host_ctr[1];
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, ctx->ev[6], ctx->ev[7]) != hipSuccess) ms = 0.f;
    ctx->st.launches += 1;
    ctx->st.kernel_ms += ms;
    ctx->st.samples += count;
    ctx->st.arcs += host_ctr[2];
    ctx->st.nodes += host_ctr[3];
    ctx->st.hyperedge_nodes += host_used <= cap ? host_used : 0;
    ctx->st.lds_bitmap = 0;
    ctx->st.slots = grid;
    if (host_used <= cap) {
      *total = host_used;
      return CENTRA_OK;
    }
    cap = host_used + 1024;   // staging overflowed: the batch is redrawn identically
  }
  return fail(ctx, CENTRA_EHIP, "sample_paths_bidir: staging did not converge");
}

}  // namespace centra
