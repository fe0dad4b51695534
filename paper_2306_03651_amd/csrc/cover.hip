// Node -> sample incidence and greedyCover(k, H) on gfx950.
//
// The incidence is the transpose of the hyperedge lists, kept as segments,
// one per batch of samples [m0, m1) appended by the progressive loop (a
// single segment for a one-off call): segment g's offsets seg_off[g][u]
// give u's entries [seg_off[g][u], seg_off[g][u+1]) of inc (sample ids) and
// inc_node (= u); a segment's entries occupy the same index range of inc as
// its hyperedges' entries do of he_nodes.  deg[u] = deg_H(u) over every
// segment.  Appending a batch costs its own entries only, so a run whose
// sample doubles builds each entry once instead of about twice.  At most
// kMaxSegments segments are kept; the next append rebuilds one segment from
// sample 0.  The order of the samples inside a row is irrelevant to every
// consumer.
//
// Greedy keeps gain[u] = number of uncovered hyperedges containing u.  A
// round is two kernels: an argmax over gain packed as (gain << 32 | ~u),
// so the maximum key is the largest gain with the lowest id, each
// workgroup writing the maximum of its slice (no atomics on one word);
// then the covering pass, whose every workgroup first reduces those
// per-workgroup maxima to the pick and then walks its share of the picked
// node's incidence row, marking each newly covered sample in a bitmap
// (atomicOr decides which thread covers it) and decrementing the gain of
// every node of that hyperedge.  All updates
// are integer, so the picks are exactly those of the sequential greedy.
// The rounds run back to back on the stream; the picked node is read from
// device memory, so no host round trip happens between rounds.
#include <mutex>
#include <string>

#include "common.hpp"
#include "internal.hpp"

namespace centra {

__global__ void k_copy_u64(const uint64_t* src, uint64_t* dst, size_t n) {
  for (size_t i = blockIdx.x * size_t(blockDim.x) + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    dst[i] = src[i];
}

static unsigned grid_for(uint64_t n, unsigned block, unsigned cap = 16384) {
  uint64_t g = (n + block - 1) / block;
  if (g > cap) g = cap;
  return g ? static_cast<unsigned>(g) : 1u;
}

// Per-workgroup aggregation of integer updates to a node-indexed array in
// an LDS hash table (open addressing, linear probing over kAggProbe slots).
// Hub nodes appear in a large fraction of the hyperedges; aggregating turns
// their per-hyperedge atomics into one global atomic per workgroup.  A node
// that finds no slot falls back to a direct global atomic.
constexpr uint32_t kAggBits = 11;
constexpr uint32_t kAggSize = 1u << kAggBits;
constexpr uint32_t kAggProbe = 8;

struct AggTable {
  uint32_t key[kAggSize];
  uint32_t cnt[kAggSize];
};

__device__ __forceinline__ void agg_init(AggTable& t) {
  for (uint32_t i = threadIdx.x; i < kAggSize; i += blockDim.x) {
    t.key[i] = kUnseen;
    t.cnt[i] = 0;
  }
}

// Adds 1 for node v; returns false if the table has no slot for v.
__device__ __forceinline__ bool agg_add(AggTable& t, uint32_t v) {
  const uint32_t h = (v * 0x9E3779B1u) >> (32 - kAggBits);
  for (uint32_t p = 0; p < kAggProbe; ++p) {
    const uint32_t slot = (h + p) & (kAggSize - 1);
    uint32_t k = t.key[slot];
    if (k == kUnseen) k = atomicCAS(&t.key[slot], kUnseen, v);
    if (k == kUnseen || k == v) {
      atomicAdd(&t.cnt[slot], 1u);
      return true;
    }
  }
  return false;
}

// Finds node v's slot (no insert); kUnseen if v has none.
__device__ __forceinline__ uint32_t agg_find(const AggTable& t, uint32_t v) {
  const uint32_t h = (v * 0x9E3779B1u) >> (32 - kAggBits);
  for (uint32_t p = 0; p < kAggProbe; ++p) {
    const uint32_t slot = (h + p) & (kAggSize - 1);
    if (t.key[slot] == v) return slot;
    if (t.key[slot] == kUnseen) return kUnseen;
  }
  return kUnseen;
}

// Transpose with per-workgroup range reservation: pass 1 counts this
// workgroup's entries per node, one atomic per node reserves a range of
// the node's row, pass 2 places the entries (the same grid-stride order in
// both passes).  Nodes without a slot reserve per entry.
// Entries go to [he_off[m0], he_off[m]) of inc; nothing is written unless
// that range lies within the `limit` entries inc holds, and no write lands
// outside it whatever the offsets (decreasing offsets raise kErrOffsets).
__global__ void k_scatter_inc_agg(const uint64_t* he_off, const uint32_t* he_nodes, uint64_t m0, uint64_t m, uint32_t n,
                                  uint64_t limit, uint64_t* cursor, uint32_t* inc, uint32_t* inc_node,
                                  uint32_t* flags) {
  __shared__ AggTable tab;
  __shared__ uint64_t base[kAggSize];
  const uint64_t I0 = he_off[m0], I1 = he_off[m];
  if (I1 > limit || I0 > I1) return;   // uniform: k_count_deg_agg raised the error
  agg_init(tab);
  __syncthreads();
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  const uint64_t s0 = m0 + blockIdx.x * uint64_t(blockDim.x) + threadIdx.x;
  for (uint64_t s = s0; s < m; s += stride) {
    const uint64_t b = he_off[s], e = he_off[s + 1];
    if (b > e) {
      atomicOr(flags, kErrOffsets);
      continue;
    }
    for (uint64_t x = b < I0 ? I0 : b; x < (e < I1 ? e : I1); ++x) {
      const uint32_t u = he_nodes[x];
      if (u < n) (void)agg_add(tab, u);
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kAggSize; i += blockDim.x) {
    if (tab.key[i] != kUnseen)
      base[i] = atomicAdd(reinterpret_cast<unsigned long long*>(&cursor[tab.key[i]]),
                          static_cast<unsigned long long>(tab.cnt[i]));
    tab.cnt[i] = 0;
  }
  __syncthreads();
  for (uint64_t s = s0; s < m; s += stride) {
    const uint64_t b = he_off[s], e = he_off[s + 1];
    if (b > e) continue;
    for (uint64_t x = b < I0 ? I0 : b; x < (e < I1 ? e : I1); ++x) {
      const uint32_t u = he_nodes[x];
      if (u >= n) continue;
      const uint32_t slot = agg_find(tab, u);
      const uint64_t p = slot != kUnseen
                             ? base[slot] + atomicAdd(&tab.cnt[slot], 1u)
                             : atomicAdd(reinterpret_cast<unsigned long long*>(&cursor[u]), 1ull);
      if (p >= I1) {   // only with decreasing offsets (flagged above)
        atomicOr(flags, kErrOffsets);
        continue;
      }
      inc[p] = static_cast<uint32_t>(s);
      inc_node[p] = u;
    }
  }
}

// deg[u] += entries of u among he_nodes[he_off[m0], he_off[m1]) (the entry
// range is read on the device; a range beyond `limit` entries counts
// nothing and raises kErrCapacity).
__global__ void k_count_deg_agg(const uint64_t* he_off, uint64_t m0, uint64_t m1, const uint32_t* he_nodes, uint32_t n,
                                uint64_t limit, uint32_t* deg, uint32_t* flags) {
  __shared__ AggTable tab;
  const uint64_t I0 = he_off[m0], I1 = he_off[m1];
  if (I1 > limit || I0 > I1) {   // uniform over the grid
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(flags, I0 > I1 ? kErrOffsets : kErrCapacity);
    return;
  }
  agg_init(tab);
  __syncthreads();
  for (uint64_t e = I0 + blockIdx.x * uint64_t(blockDim.x) + threadIdx.x; e < I1; e += uint64_t(gridDim.x) * blockDim.x) {
    const uint32_t u = he_nodes[e];
    if (u >= n) {
      atomicOr(flags, kErrNodeRange);
      continue;
    }
    if (!agg_add(tab, u)) atomicAdd(&deg[u], 1u);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kAggSize; i += blockDim.x)
    if (tab.key[i] != kUnseen) atomicAdd(&deg[tab.key[i]], tab.cnt[i]);
}

__global__ void k_add_u32_to(const uint32_t* a, uint32_t n, uint32_t* acc) {
  for (uint32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < n; u += gridDim.x * blockDim.x) acc[u] += a[u];
}

// a[i] += *add for i < n (the addend read on the device).
__global__ void k_offset_u64(uint64_t* a, uint64_t n, const uint64_t* add) {
  const uint64_t x = *add;
  if (x == 0) return;
  for (uint64_t i = blockIdx.x * uint64_t(blockDim.x) + threadIdx.x; i < n; i += uint64_t(gridDim.x) * blockDim.x)
    a[i] += x;
}

// Launches the build of one incidence segment: samples [m0, m1), whose
// entries [he_off[m0], he_off[m1]) of he_nodes are located on the device
// (span_cap bounds their number, for the launch shapes only; inc and
// inc_node hold `limit` entries, and a segment reaching beyond them is
// left empty with kErrCapacity raised); its offsets go to `off` (absolute
// into inc), its degrees to sdeg, and deg accumulates them (cleared first
// when `first_segment`).  Launches only.
void incidence_segment(uint32_t n, uint64_t m0, uint64_t m1, uint64_t span_cap, uint64_t limit, const uint64_t* he_off,
                       const uint32_t* he_nodes, bool first_segment, uint32_t* deg, uint32_t* sdeg, uint64_t* off,
                       uint64_t* cur, uint32_t* inc, uint32_t* inc_node, uint64_t* scan_tiles, uint32_t* flags,
                       hipStream_t s) {
  if (first_segment) fill_u32(deg, 0, n, s);
  fill_u32(sdeg, 0, n, s);
  if (m1 > m0 && span_cap)
    hipLaunchKernelGGL(k_count_deg_agg, dim3(grid_for(span_cap, 256, 2048)), dim3(256), 0, s, he_off, m0, m1, he_nodes, n,
                       limit, sdeg, flags);
  excl_scan_u32_to_u64_ws(sdeg, off, n, scan_tiles, s);
  if (m0) hipLaunchKernelGGL(k_offset_u64, dim3(grid_for(uint64_t(n) + 1, 256)), dim3(256), 0, s, off, uint64_t(n) + 1,
                             he_off + m0);
  hipLaunchKernelGGL(k_copy_u64, dim3(grid_for(n, 256)), dim3(256), 0, s, off, cur, size_t(n));
  if (m1 > m0)
    hipLaunchKernelGGL(k_scatter_inc_agg, dim3(grid_for(m1 - m0, 256, 2048)), dim3(256), 0, s, he_off, he_nodes, m0, m1,
                       n, limit, cur, inc, inc_node, flags);
  hipLaunchKernelGGL(k_add_u32_to, dim3(grid_for(n, 256)), dim3(256), 0, s, sdeg, n, deg);
}

int build_incidence(centra_ctx* ctx, uint32_t n, uint64_t m0, uint64_t m1, const uint64_t* he_off,
                    const uint32_t* he_nodes, hipStream_t s, uint64_t entry_cap) {
  ctx->ext_inc = false;   // the extend calls' state is valid only after their own builds
  if (m0 == 0 || ctx->inc_nseg >= kMaxSegments) {   // a new sample, or too many segments: start over
    ctx->inc_nseg = 0;
    m0 = 0;
  }
  uint64_t I0 = 0, I1 = entry_cap;
  if (entry_cap == ~0ull) {   // sizes read from the device (one synchronisation)
    uint64_t ends[2] = {0, 0};
    CENTRA_HIP(ctx, hipMemcpyAsync(&ends[0], he_off + m0, 8, hipMemcpyDeviceToHost, s));
    CENTRA_HIP(ctx, hipMemcpyAsync(&ends[1], he_off + m1, 8, hipMemcpyDeviceToHost, s));
    CENTRA_HIP(ctx, hipStreamSynchronize(s));
    I0 = ends[0];
    I1 = ends[1];
  }
  const uint32_t g = ctx->inc_nseg;
  int rc;
  if ((rc = ensure(ctx, ctx->deg, size_t(n) * 4, g > 0, s))) return rc;
  if ((rc = ensure(ctx, ctx->seg_deg, size_t(n) * 4, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->inc_off, (size_t(g) + 1) * (size_t(n) + 1) * 8, g > 0, s))) return rc;
  if ((rc = ensure(ctx, ctx->inc_cursor, size_t(n) * 8, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->inc, (I1 ? I1 : 1) * 4, g > 0, s))) return rc;
  if ((rc = ensure(ctx, ctx->inc_node, (I1 ? I1 : 1) * 4, g > 0, s))) return rc;
  if ((rc = ensure(ctx, ctx->scan_tmp, scan_tile_words(n) * 8, false, s))) return rc;
  if (n <= kIncBucketMaxNodes) {
    if ((rc = ensure(ctx, ctx->inc_ws, incidence_ws_bytes(n, I1 - I0), false, s))) return rc;
    incidence_segment_bucketed(n, m0, m1, I1 - I0, I1, he_off, he_nodes, g == 0, static_cast<uint32_t*>(ctx->deg.ptr),
                               static_cast<uint32_t*>(ctx->seg_deg.ptr),
                               static_cast<uint64_t*>(ctx->inc_off.ptr) + size_t(g) * (size_t(n) + 1),
                               static_cast<uint64_t*>(ctx->inc_cursor.ptr), static_cast<uint32_t*>(ctx->inc.ptr),
                               static_cast<uint32_t*>(ctx->inc_node.ptr), ctx->inc_ws.ptr, ctx->d_flags, s);
  } else {
    incidence_segment(n, m0, m1, I1 - I0, I1, he_off, he_nodes, g == 0, static_cast<uint32_t*>(ctx->deg.ptr),
                      static_cast<uint32_t*>(ctx->seg_deg.ptr),
                      static_cast<uint64_t*>(ctx->inc_off.ptr) + size_t(g) * (size_t(n) + 1),
                      static_cast<uint64_t*>(ctx->inc_cursor.ptr), static_cast<uint32_t*>(ctx->inc.ptr),
                      static_cast<uint32_t*>(ctx->inc_node.ptr), static_cast<uint64_t*>(ctx->scan_tmp.ptr), ctx->d_flags,
                      s);
  }
  CENTRA_HIP(ctx, hipGetLastError());
  ctx->inc_nseg = g + 1;
  ++ctx->inc_gen;
  ctx->inc_m0 = m0;
  ctx->inc_span_cap = I1 - I0;
  ctx->inc_m1 = m1;
  ctx->inc_limit = I1;
  if (ctx->inc_seg_m0.size() < size_t(g) + 1) ctx->inc_seg_m0.resize(size_t(g) + 1);
  ctx->inc_seg_m0[g] = m0;
  return CENTRA_OK;
}

int incidence_reserve(centra_ctx* ctx, uint32_t n, uint64_t entries, uint32_t segments, hipStream_t s) {
  int rc;
  if ((rc = ensure(ctx, ctx->deg, size_t(n) * 4, true, s))) return rc;
  if ((rc = ensure(ctx, ctx->seg_deg, size_t(n) * 4, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->inc_off, (size_t(segments) + 1) * (size_t(n) + 1) * 8, true, s))) return rc;
  if ((rc = ensure(ctx, ctx->inc_cursor, size_t(n) * 8, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->inc, (entries ? entries : 1) * 4, true, s))) return rc;
  if ((rc = ensure(ctx, ctx->inc_node, (entries ? entries : 1) * 4, true, s))) return rc;
  if (n <= kIncBucketMaxNodes && (rc = ensure(ctx, ctx->inc_ws, incidence_ws_bytes(n, entries), false, s))) return rc;
  return ensure(ctx, ctx->scan_tmp, scan_tile_words(n) * 8, false, s);
}

// ---------------------------------------------------------------------------
__global__ void k_gain_init(const uint32_t* deg, uint32_t n, int32_t* gain) {
  for (uint32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < n; u += gridDim.x * blockDim.x)
    gain[u] = static_cast<int32_t>(deg[u]);
}

constexpr int kArgBlock = 256;

constexpr unsigned kArgGrid = 512;   // workgroups of the argmax (and per-workgroup maxima)

constexpr int kArgUnroll = 4;       // 4-node groups a thread loads at once

__device__ __forceinline__ uint64_t gain_key(int32_t g, uint32_t u) {
  return g > 0 ? (static_cast<uint64_t>(g) << 32) | (0xFFFFFFFFu - u) : 0ull;
}

// The largest key (gain << 32 | ~u, 0 if no positive gain) of the slice
// of workgroup b of nb: the 4-node groups b*kArgBlock + i*nb*kArgBlock
// (gain is 16-byte aligned), kArgUnroll groups per thread loaded together
// so that their round trips overlap; workgroup 0 also takes the n % 4
// nodes past the last group.  The maximum of the keys does not depend on
// how the nodes are split.
__device__ __forceinline__ uint64_t argmax_slice(const int32_t* gain, uint32_t n, uint32_t b, uint32_t nb,
                                                 uint64_t* red) {
  uint64_t key = 0;
  const uint32_t nv = n >> 2;
  const int4* g4 = reinterpret_cast<const int4*>(gain);
  const uint32_t stride = nb * kArgBlock;
  for (uint32_t w = b * kArgBlock + threadIdx.x; w < nv; w += kArgUnroll * stride) {
    int4 x[kArgUnroll];
#pragma unroll
    for (int j = 0; j < kArgUnroll; ++j) {
      const uint32_t wj = w + j * stride;
      x[j] = wj < nv ? g4[wj] : make_int4(0, 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < kArgUnroll; ++j) {
      const uint32_t u = (w + j * stride) * 4;   // groups past nv hold zeros: key 0
      uint64_t k = gain_key(x[j].x, u);
      k = max(k, gain_key(x[j].y, u + 1));
      k = max(k, gain_key(x[j].z, u + 2));
      k = max(k, gain_key(x[j].w, u + 3));
      key = max(key, k);
    }
  }
  if (b == 0 && threadIdx.x < (n & 3u)) {
    const uint32_t u = (nv << 2) + threadIdx.x;
    key = max(key, gain_key(gain[u], u));
  }
  return block_max_u64<kArgBlock>(key, red);
}

// part[b] = the largest key of the slice of workgroup b (0 if the slice has
// no positive gain)
__global__ __launch_bounds__(kArgBlock) void k_argmax(const int32_t* gain, uint32_t n, uint64_t* part) {
  __shared__ uint64_t red[kArgBlock / kWave];
  const uint64_t key = argmax_slice(gain, n, blockIdx.x, gridDim.x, red);
  if (threadIdx.x == 0) part[blockIdx.x] = key;
}

constexpr int kCoverBlock = 256;

// LDS of a covering walk.
struct CoverShared {
  AggTable tab;
  uint64_t red[kCoverBlock / kWave];
  uint64_t seg_beg[kMaxSegments], seg_pre[kMaxSegments + 1];
  uint32_t scan[kCoverBlock / kWave + 1];
  uint64_t hbeg[kCoverBlock];  // he_off of the step's newly covered samples
  uint32_t hoff[kCoverBlock];  // exclusive prefix of their hyperedge sizes
};

// The walk of one covering pass, workgroup b of nb, for the pick u: its
// share of u's incidence rows in the n_seg segments walked as one row
// (their concatenation), one entry per thread per step.  A step marks the
// newly covered samples among its entries, then the workgroup decrements
// the gains of all their nodes together (the concatenation of their
// hyperedges split evenly over the threads), so long hyperedges (paths of
// thousands of nodes) are spread over the workgroup instead of walked by
// one thread.
__device__ __forceinline__ void cover_walk(uint32_t u, const uint64_t* seg_off, uint32_t n_seg, const uint32_t* inc,
                                           const uint64_t* he_off, const uint32_t* he_nodes, uint32_t n,
                                           uint32_t* covered, int32_t* gain, uint64_t* newcov, uint32_t b, uint32_t nb,
                                           CoverShared& sh) {
  if (threadIdx.x < kWave) {   // segment starts and the prefix of the row lengths (n_seg <= 64)
    const uint32_t g = threadIdx.x;
    uint64_t rb = 0, len = 0;
    if (g < n_seg) {
      const uint64_t* o = seg_off + size_t(g) * (size_t(n) + 1);
      rb = o[u];
      len = o[u + 1] - rb;
    }
    const uint64_t incl = wave_incl_scan_u64(len);
    if (g < n_seg) {
      sh.seg_beg[g] = rb;
      sh.seg_pre[g + 1] = incl;
    }
    if (g == 0) sh.seg_pre[0] = 0;
  }
  __syncthreads();
  const uint64_t row = sh.seg_pre[n_seg];
  const uint64_t lead = b * uint64_t(kCoverBlock);
  if (lead >= row) {   // uniform per workgroup: nothing of the row lands here
    __syncthreads();   // seg_* are reused by the caller's next item
    return;
  }
  agg_init(sh.tab);
  __syncthreads();
  uint64_t cnt = 0;
  uint32_t g = 0;
  const uint64_t stride = uint64_t(nb) * kCoverBlock;
  for (uint64_t base = lead; base < row; base += stride) {   // uniform trip count
    const uint64_t q = base + threadIdx.x;
    uint32_t len = 0;
    uint64_t h0 = 0;
    if (q < row) {
      while (q >= sh.seg_pre[g + 1]) ++g;
      const uint32_t s = inc[sh.seg_beg[g] + (q - sh.seg_pre[g])];
      // the hyperedge's bounds are loaded before the covering atomic
      // returns, so the two round trips overlap
      h0 = he_off[s];
      const uint64_t h1 = he_off[s + 1];
      const uint32_t bit = 1u << (s & 31u);
      const uint32_t old = atomicOr(&covered[s >> 5], bit);
      if (!(old & bit)) {   // newly covered
        ++cnt;
        len = static_cast<uint32_t>(h1 - h0);
      }
    }
    uint32_t total;
    const uint32_t off = block_excl_scan_u32<kCoverBlock>(len, &total, sh.scan);
    sh.hbeg[threadIdx.x] = h0;
    sh.hoff[threadIdx.x] = off;
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < total; e += kCoverBlock) {
      // the sample holding entry e: the last i with hoff[i] <= e and a
      // nonempty hyperedge (empty ones repeat their successor's offset)
      int lo = 0, hi = kCoverBlock - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sh.hoff[mid] <= e)
          lo = mid;
        else
          hi = mid - 1;
      }
      const uint32_t v = he_nodes[sh.hbeg[lo] + (e - sh.hoff[lo])];
      if (v < n && !agg_add(sh.tab, v)) atomicSub(&gain[v], 1);
    }
    __syncthreads();
  }
  cnt = block_sum_u64<kCoverBlock>(cnt, sh.red);   // contains the barrier before the flush
  for (uint32_t i = threadIdx.x; i < kAggSize; i += kCoverBlock)
    if (sh.tab.key[i] != kUnseen) atomicSub(&gain[sh.tab.key[i]], static_cast<int32_t>(sh.tab.cnt[i]));
  if (threadIdx.x == 0 && cnt) atomicAdd(reinterpret_cast<unsigned long long*>(newcov), cnt);
  __syncthreads();   // the table and seg_* are reused by the caller's next item
}

// One covering pass, workgroup b of nb: reduces the n_part per-workgroup
// maxima to the round's pick (workgroup 0 writes it to *best), then walks
// its share of the pick's rows.
__device__ __forceinline__ void cover_pass(const uint64_t* part, uint32_t n_part, uint64_t* best, const uint64_t* seg_off,
                                           uint32_t n_seg, const uint32_t* inc, const uint64_t* he_off,
                                           const uint32_t* he_nodes, uint32_t n, uint32_t* covered, int32_t* gain,
                                           uint64_t* newcov, uint32_t b, uint32_t nb, CoverShared& sh) {
  static_assert(kArgGrid <= 2 * kCoverBlock, "two maxima per thread");
  const uint64_t p0 = threadIdx.x < n_part ? part[threadIdx.x] : 0ull;
  const uint64_t p1 = threadIdx.x + kCoverBlock < n_part ? part[threadIdx.x + kCoverBlock] : 0ull;
  const uint64_t key = block_max_u64<kCoverBlock>(p0 > p1 ? p0 : p1, sh.red);
  if (b == 0 && threadIdx.x == 0) *best = key;
  if ((key >> 32) == 0) return;
  cover_walk(0xFFFFFFFFu - static_cast<uint32_t>(key), seg_off, n_seg, inc, he_off, he_nodes, n, covered, gain, newcov,
             b, nb, sh);
}

// best = the round's pick (written by workgroup 0): the largest of the
// n_part per-workgroup maxima of the argmax.
__global__ __launch_bounds__(kCoverBlock) void k_cover(const uint64_t* part, uint32_t n_part, uint64_t* best,
                                                       const uint64_t* seg_off, uint32_t n_seg, const uint32_t* inc,
                                                       const uint64_t* he_off, const uint32_t* he_nodes, uint32_t n,
                                                       uint32_t* covered, int32_t* gain, uint64_t* newcov) {
  __shared__ CoverShared sh;
  cover_pass(part, n_part, best, seg_off, n_seg, inc, he_off, he_nodes, n, covered, gain, newcov, blockIdx.x, gridDim.x,
             sh);
}

// ---------------------------------------------------------------------------
// Greedy in batches of picks.  A round of two kernels is a chain of dependent
// trips to memory, 21 us however few samples it covers (n = m = 10^6), and
// greedy needs k of them in sequence.  But the picks that follow one another
// mostly come from the few nodes of largest gain, and while one of those is
// the best of all, the rounds depend on nothing but the samples that several
// of them share.  So a batch
//   1. finds up to 64 candidates, the nodes of largest gain, and tau, the
//      largest key (gain << 32 | ~u) of any other node;
//   2. sets, for every uncovered sample of their rows, the bits of the
//      candidates it holds in a mask of the sample, and lists the masks of two
//      bits or more;
//   3. runs greedy rounds over the candidates in one workgroup: a candidate's
//      gain only falls by the listed masks it shares with a pick.  Gains only
//      fall, so as long as the best candidate's key exceeds tau, it is the
//      largest of all nodes': the sequential greedy's pick;
//   4. covers the picks' rows at once (the order of covering changes no gain).
// The first round's pick always is a candidate, so a batch has at least one;
// two batches make 50 picks on the hyperedge sets and path samples measured.
// The host reads how far a batch came and starts another, or, where batches
// yield little, goes on by rounds.  n = m = 10^6, 4M entries, k = 50: 1,040 us
// by rounds, 270 in batches; BA n = 10^5, 400,000 path samples, k = 50: 650 by
// rounds, 280 in batches.
constexpr uint32_t kCands = 64;
constexpr uint32_t kTopBlocks = 64, kTopBlock = 256, kTopCols = kTopBlocks * kTopBlock;
constexpr uint32_t kBatchBlock = 1024;
constexpr uint32_t kBatchSegs = 16;            // incidence segments at most
constexpr uint32_t kBatchRows = kCands * kBatchSegs;
constexpr uint32_t kBatchList = 1u << 19;      // masks listed at most
constexpr uint32_t kBatchMinK = 12;            // rounds from which batches pay
// Samples up to which they do: one workgroup goes through the listed masks for
// every pick, and their number grows with m (a whole run on BA n = 10^5 up to
// 400,000 samples: 9.4 ms in batches, 10.8 by rounds; build and greedy of 4M
// samples of BA n = 10^6: 3.7 in batches, 2.3 by rounds).
constexpr uint64_t kBatchMaxM = 2u << 20;
constexpr uint32_t kBatchMinPicks = 8;         // a batch with fewer is the last
// A batch reads all its candidates' rows, a round its pick's alone, so batches
// pay while the rows are short against the rounds spared: entries per round
// (us, k = 50, rounds / batches: BA n = 10^5, 400,000 path samples, 321,000
// entries: 853 / 714, 800,000 samples, 645,000 entries: 985 / 1,115; synthetic, n
// = 200,000, 500,000 samples of 16, 499,000: 2,002 / 1,578; n = 20,000, 10^6 of
// 4, 573,000: 1,250 / 1,135; n = 2,000, 500,000 of 4, 593,000: 1,074 / 1,226; k =
// 12, BA, 80,000: 325 / 310, 321,000: 418 / 519).
constexpr uint64_t kBatchEntries = 12288;
// And the candidates must not overlap so much that few of them stay above tau:
// entries per sample, over the 64 of them (k = 50: n = 2,000, 50,000 samples of 4
// nodes, 1.2: 622 / 435; n = 200,000, 200,000 of 16, 1.0: 1,610 / 899; n = 20,000,
// 200,000 of 16, 2.1: 1,169 / 1,283; n = 8,000, 20,000 of 64, 9.4: 824 / 923).
constexpr uint64_t kBatchOverlap = 2;

// Device state of a batch.  Row i = c * n_seg + g is candidate c's in segment
// g; pre is the prefix of the rows' lengths.
struct BatchState {
  uint64_t tau;
  uint32_t r;          // rounds done
  uint32_t fail;       // a node twice in a hyperedge, more masks than the list holds, or rows too long
  uint32_t done;       // no positive gain is left
  uint32_t n_cand, n_list, pad;
  uint32_t node[kCands];
  int32_t gain[kCands];
  uint64_t chosen;     // bits of the candidates that were picked
  uint64_t beg[kBatchRows], pre[kBatchRows + 1];
};

struct BatchArgs {
  uint32_t n, n_seg, k, r;   // r: rounds done before
  uint64_t m;
  const uint64_t* seg_off;
  const uint32_t* inc;
  const uint64_t* he_off;
  const uint32_t* he_nodes;
  int32_t* gain;
  uint32_t* covered;
  uint64_t* best;     // u64[k] keys
  uint64_t* newcov;   // u64[k]
  uint64_t* part;     // u64[kTopCols + kTopBlocks]
  BatchState* st;
  uint64_t* list;     // u64[kBatchList]
  uint64_t* mask;     // u64[m]
};

// Bin of a positive gain: 8 bins per bit length, by the 3 bits below the
// leading one (nondecreasing in g).  (The engine's lists use it too.)
constexpr uint32_t kGainBins = 256;
__device__ __forceinline__ uint32_t gain_bin(uint32_t g) {
  const uint32_t bl = 32u - __clz(g);
  const uint32_t sub = bl >= 4 ? (g >> (bl - 4)) & 7u : (g << (4 - bl)) & 7u;
  return (bl - 1) * 8 + sub;
}

// The last row that starts at or before entry e.
__device__ __forceinline__ uint32_t batch_row(const uint64_t* pre, uint64_t e) {
  uint32_t i = 0;
#pragma unroll
  for (uint32_t step = kBatchRows / 2; step; step >>= 1)
    if (pre[i + step] <= e) i += step;
  return i;
}

// Calls f(sample, candidate) for every entry of the candidates' rows.
template <typename F>
__device__ __forceinline__ void batch_entries(const BatchArgs& a, uint64_t* pre, const F& f) {
  for (uint32_t i = threadIdx.x; i <= kBatchRows; i += blockDim.x) pre[i] = a.st->pre[i];
  __syncthreads();
  const uint64_t total = pre[kBatchRows];
  for (uint64_t e0 = uint64_t(blockIdx.x) * blockDim.x; e0 < total; e0 += uint64_t(gridDim.x) * blockDim.x) {
    const uint64_t e = e0 + threadIdx.x;
    if (e >= total) continue;
    const uint32_t i = batch_row(pre, e);
    f(a.inc[a.st->beg[i] + (e - pre[i])], i / a.n_seg);
  }
}

// part[x] = the largest key of the nodes u = x mod kTopCols (nodes of large
// gain often are neighbours by id: that spreads them), part[kTopCols + b] the
// largest of the second keys of workgroup b's columns.
// Masks that the batch before set are cleared.
__global__ __launch_bounds__(kTopBlock) void k_batch_top(BatchArgs a, int first) {
  __shared__ uint64_t red[kTopBlock / kWave];
  __shared__ uint64_t pre[kBatchRows + 1];
  if (!first) batch_entries(a, pre, [&](uint32_t s, uint32_t) { a.mask[s] = 0; });
  constexpr int kLoads = 16;
  const uint32_t x = blockIdx.x * kTopBlock + threadIdx.x;
  uint64_t k1 = 0, k2 = 0;
  for (uint64_t u0 = x; u0 < a.n; u0 += uint64_t(kLoads) * kTopCols) {
    int32_t g[kLoads];
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const uint64_t u = u0 + uint64_t(j) * kTopCols;
      g[j] = u < a.n ? a.gain[u] : 0;
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const uint64_t key = gain_key(g[j], static_cast<uint32_t>(u0) + j * kTopCols);
      const uint64_t low = key < k1 ? key : k1;
      k1 = key > k1 ? key : k1;
      k2 = low > k2 ? low : k2;
    }
  }
  a.part[x] = k1;
  k2 = block_max_u64<kTopBlock>(k2, red);
  if (threadIdx.x == 0) a.part[kTopCols + blockIdx.x] = k2;
}

// The candidates: the largest of the columns' keys, and of the others those
// of the bins of gains that fit; tau; the candidates' rows.
__global__ __launch_bounds__(kBatchBlock) void k_batch_cands(BatchArgs a) {
  __shared__ uint64_t red[2 * Coll<kBatchBlock>::kHalf];
  __shared__ uint32_t hist[kGainBins], cut, used;
  __shared__ uint32_t node[kCands];
  Coll<kBatchBlock> co{red, 0};
  constexpr uint32_t kOwn = kTopCols / kBatchBlock;
  const uint32_t tid = threadIdx.x;
  uint64_t key[kOwn], mx = 0, tau = tid < kTopBlocks ? a.part[kTopCols + tid] : 0ull;
#pragma unroll
  for (uint32_t i = 0; i < kOwn; ++i) key[i] = a.part[i * kBatchBlock + tid];
  if (tid < kGainBins) hist[tid] = 0;
  if (tid < kCands) node[tid] = kUnseen;
  if (tid == 0) used = 1;   // place 0 is the largest's
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kOwn; ++i) {
    if (key[i]) atomicAdd(&hist[gain_bin(static_cast<uint32_t>(key[i] >> 32))], 1u);
    mx = key[i] > mx ? key[i] : mx;
  }
  mx = co.max(mx);
  if (tid < kWave) {
    // the lowest bin that, with those above it, holds at most kCands keys
    // (the top one in any case: what does not fit counts for tau)
    uint32_t h[kGainBins / kWave], sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < kGainBins / kWave; ++j) {
      h[j] = hist[kGainBins - 1 - (tid * (kGainBins / kWave) + j)];
      sum += h[j];
    }
    uint32_t run = wave_incl_scan_u32(sum) - sum, fit = 0;
#pragma unroll
    for (uint32_t j = 0; j < kGainBins / kWave; ++j) {
      run += h[j];
      fit += run <= kCands ? 1u : 0u;
    }
    fit = wave_sum_u32(fit);   // bins from the top that fit together
    if (tid == 0) {
      const uint32_t top = mx ? gain_bin(static_cast<uint32_t>(mx >> 32)) : 0u;
      const uint32_t lowest = kGainBins - fit;
      cut = lowest < top ? lowest : top;
    }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kOwn; ++i) {
    if (!key[i]) continue;
    uint32_t at = kCands;
    if (key[i] == mx)
      at = 0;
    else if (gain_bin(static_cast<uint32_t>(key[i] >> 32)) >= cut)
      at = atomicAdd(&used, 1u);
    if (at < kCands) {
      node[at] = 0xFFFFFFFFu - static_cast<uint32_t>(key[i]);
      a.st->node[at] = node[at];
      a.st->gain[at] = static_cast<int32_t>(key[i] >> 32);
    } else {
      tau = key[i] > tau ? key[i] : tau;
    }
  }
  tau = co.max(tau);
  const uint32_t n_cand = mx ? (used < kCands ? used : kCands) : 0u, rows = n_cand * a.n_seg;   // (rows <= kBatchBlock)
  uint64_t rb = 0, len = 0, total;
  if (tid < rows) {
    const uint64_t* o = a.seg_off + size_t(tid % a.n_seg) * (size_t(a.n) + 1) + node[tid / a.n_seg];
    rb = o[0];
    len = o[1] - rb;
  }
  const uint64_t before = co.scan(len, &total);
  a.st->beg[tid] = rb;
  a.st->pre[tid] = before;
  if (tid == 0) {
    const bool fail = total > kBatchEntries * (a.k - a.r) || total > kBatchOverlap * a.m;
    a.st->pre[kBatchRows] = fail ? 0 : total;   // (then there is nothing to read)
    if (fail) a.st->fail = 1;
    a.st->tau = tau;
    a.st->n_cand = n_cand;
    a.st->n_list = 0;
    a.st->done = mx ? 0u : 1u;
  }
}

__global__ __launch_bounds__(256) void k_batch_mask(BatchArgs a) {
  __shared__ uint64_t pre[kBatchRows + 1];
  batch_entries(a, pre, [&](uint32_t s, uint32_t c) {
    if (a.covered[s >> 5] >> (s & 31u) & 1u) return;
    const uint64_t old = atomicOr(reinterpret_cast<unsigned long long*>(&a.mask[s]), 1ull << c);
    if (old >> c & 1ull) a.st->fail = 1;
  });
}

// (One addition to the list's length per workgroup and step: one per wave took
// 19 us for 130,000 entries, the additions to one word in a row.)
__global__ __launch_bounds__(256) void k_batch_list(BatchArgs a) {
  __shared__ uint64_t pre[kBatchRows + 1], red[2 * Coll<256>::kHalf];
  __shared__ uint32_t base;
  Coll<256> co{red, 0};
  for (uint32_t i = threadIdx.x; i <= kBatchRows; i += 256) pre[i] = a.st->pre[i];
  __syncthreads();
  const uint64_t total = pre[kBatchRows];
  for (uint64_t e0 = uint64_t(blockIdx.x) * 256; e0 < total; e0 += uint64_t(gridDim.x) * 256) {   // uniform
    const uint64_t e = e0 + threadIdx.x;
    uint64_t w = 0;
    if (e < total) {
      const uint32_t i = batch_row(pre, e);
      w = a.mask[a.inc[a.st->beg[i] + (e - pre[i])]];
      // two bits at least, and the lowest candidate's entry
      if ((w & (w - 1)) == 0 || (w & (0ull - w)) != 1ull << (i / a.n_seg)) w = 0;
    }
    uint64_t found;
    const uint32_t at = static_cast<uint32_t>(co.scan(w ? 1u : 0u, &found));
    if (found && threadIdx.x == 0) base = atomicAdd(&a.st->n_list, static_cast<uint32_t>(found));
    __syncthreads();
    if (w) {
      if (base + at < kBatchList)
        a.list[base + at] = w;
      else
        a.st->fail = 1;
    }
    __syncthreads();
  }
}

// The rounds over the candidates.  Thread t owns the masks t, t + 1024, ... of
// the list and drops those that a pick covers.
__global__ __launch_bounds__(kBatchBlock) void k_batch_solve(BatchArgs a) {
  __shared__ int32_t gain[kCands];
  __shared__ uint32_t node[kCands];
  __shared__ uint32_t pick;
  const uint32_t tid = threadIdx.x;
  if (tid < kCands) {
    const bool is = tid < a.st->n_cand;
    gain[tid] = is ? a.st->gain[tid] : 0;
    node[tid] = is ? a.st->node[tid] : 0u;
  }
  const uint32_t n_list = a.st->n_list;
  uint32_t own = a.st->fail || tid >= n_list ? 0u : (n_list - tid + kBatchBlock - 1) / kBatchBlock;
  uint32_t r = a.st->r;
  uint64_t chosen = 0;
  const uint64_t tau = a.st->tau;
  const bool run = !a.st->fail;
  __syncthreads();
  while (run && r < a.k) {
    if (tid < kWave) {
      const uint64_t key = gain_key(gain[tid], node[tid]);
      const uint64_t mx = wave_max_u64(key);
      if (key == mx && mx > tau) {   // one lane: keys are distinct, mx > 0
        pick = tid;
        a.best[r] = key;
        a.newcov[r] = key >> 32;
        gain[tid] = 0;
      }
      if (mx <= tau) {
        pick = kCands;
        if (tau == 0 && tid == 0) a.st->done = 1;   // (mx is 0 too: no gain is left anywhere)
      }
    }
    __syncthreads();
    const uint32_t c = pick;
    if (c == kCands) break;
    uint32_t kept = 0;
    constexpr uint32_t kLoads = 8;   // masks under way at once
    for (uint32_t i = 0; i < own; i += kLoads) {
      uint64_t x[kLoads];
#pragma unroll
      for (uint32_t j = 0; j < kLoads; ++j) x[j] = i + j < own ? a.list[size_t(i + j) * kBatchBlock + tid] : 0ull;
#pragma unroll
      for (uint32_t j = 0; j < kLoads; ++j) {
        uint64_t m = x[j];
        if (m >> c & 1ull) {
          for (m &= ~(1ull << c); m; m &= m - 1)
            atomicSub(&gain[__ffsll(static_cast<unsigned long long>(m)) - 1], 1);
        } else if (m) {
          if (kept != i + j) a.list[size_t(kept) * kBatchBlock + tid] = m;   // (at or below the places read)
          ++kept;
        }
      }
    }
    own = kept;
    ++r;
    chosen |= 1ull << c;
    __syncthreads();
  }
  if (tid == 0) {
    a.st->r = r;
    a.st->chosen = chosen;
  }
}

// Covers the picks' rows.  A sample is covered by the entry of its first pick
// (its mask says which), so no thread needs the answer of an atomic.  A
// hyperedge of up to kShort nodes is walked by that entry's thread; longer
// ones (paths of thousands of nodes) by the workgroup, the concatenation of
// the step's split evenly over the threads.
__global__ __launch_bounds__(kCoverBlock) void k_batch_cover(BatchArgs a) {
  constexpr uint32_t kShort = 8;
  __shared__ AggTable tab;
  __shared__ uint64_t pre[kBatchRows + 1], hbeg[kCoverBlock];
  __shared__ uint32_t hoff[kCoverBlock], scan[kCoverBlock / kWave + 1];
  for (uint32_t i = threadIdx.x; i <= kBatchRows; i += kCoverBlock) pre[i] = a.st->pre[i];
  agg_init(tab);
  const uint64_t chosen = a.st->chosen;
  __syncthreads();
  const uint64_t total_e = chosen ? pre[kBatchRows] : 0ull;
  const uint64_t stride = uint64_t(gridDim.x) * kCoverBlock;
  for (uint64_t e0 = uint64_t(blockIdx.x) * kCoverBlock; e0 < total_e; e0 += stride) {   // uniform trip count
    const uint64_t e = e0 + threadIdx.x;
    uint32_t len = 0;
    uint64_t h0 = 0;
    const uint32_t i = e < total_e ? batch_row(pre, e) : 0u;
    if (e < total_e && chosen >> (i / a.n_seg) & 1ull) {
      const uint32_t s = a.inc[a.st->beg[i] + (e - pre[i])];
      const uint64_t w = a.mask[s] & chosen;
      if ((w & (0ull - w)) == 1ull << (i / a.n_seg)) {
        h0 = a.he_off[s];
        len = static_cast<uint32_t>(a.he_off[s + 1] - h0);
        atomicOr(&a.covered[s >> 5], 1u << (s & 31u));
        if (len <= kShort) {
          uint32_t v[kShort];
#pragma unroll
          for (uint32_t j = 0; j < kShort; ++j) v[j] = j < len ? a.he_nodes[h0 + j] : kUnseen;
#pragma unroll
          for (uint32_t j = 0; j < kShort; ++j)
            if (v[j] < a.n && !agg_add(tab, v[j])) atomicSub(&a.gain[v[j]], 1);
          len = 0;
        }
      }
    }
    if (!__syncthreads_or(len != 0)) continue;
    uint32_t total;
    const uint32_t off = block_excl_scan_u32<kCoverBlock>(len, &total, scan);
    hbeg[threadIdx.x] = h0;
    hoff[threadIdx.x] = off;
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < total; x += kCoverBlock) {
      // the sample holding entry x: the last i with hoff[i] <= x (the others,
      // without nodes to walk, repeat their successor's offset)
      uint32_t l = 0;
#pragma unroll
      for (uint32_t step = kCoverBlock / 2; step; step >>= 1)
        if (hoff[l + step] <= x) l += step;
      const uint32_t v = a.he_nodes[hbeg[l] + (x - hoff[l])];
      if (v < a.n && !agg_add(tab, v)) atomicSub(&a.gain[v], 1);
    }
    __syncthreads();
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kAggSize; i += kCoverBlock)
    if (tab.key[i] != kUnseen) atomicSub(&a.gain[tab.key[i]], static_cast<int32_t>(tab.cnt[i]));
}

// ---------------------------------------------------------------------------
// Greedy of many queries at once (the engine's fused rounds): blockIdx.y
// selects the query's descriptor; a query whose k is reached, or that is
// inactive (k = 0), leaves its workgroups at once.  The round number comes
// from device memory (round_base[0] + r_local), so a captured sequence of
// rounds can be replayed for the next rounds after the base is advanced.
//
// Candidate lists.  Gains only decrease, so once every node of gain >= tau
// has been collected into a list, every node outside the list stays below
// tau; while the list's largest gain is >= tau, the argmax over the list
// (largest gain, lowest id) is the argmax over all nodes, and a round reads
// the list's gains instead of all n.  A query cycles through three modes,
// decided after each round from device state:
//   full     every workgroup scans its slice of all n gains and adds a
//            histogram of them (8 bins per octave); after the round, tau is
//            the lowest bin bound whose bins and those above hold at most
//            kCandMax nodes (if any);
//   compact  a full scan that also appends every node of gain >= tau to the
//            list (at most kCandMax: gains were at most the histogram's);
//   list     one workgroup scans the list.
// The round after a list's largest gain falls below tau is full again.
constexpr uint32_t kCandMax = 8192;
constexpr uint32_t kModeFull = 0, kModeCompact = 1, kModeList = 2;

// Smallest gain of bin b (or of the next nonempty bin above it).
__device__ __forceinline__ uint32_t bin_min(uint32_t b) {
  const uint32_t bl = b / 8 + 1, sub = b % 8;
  if (bl >= 4) return (8u + sub) << (bl - 4);
  for (uint32_t g = 1; g < 16; ++g)
    if (gain_bin(g) >= b) return g;
  return 16;
}

__global__ __launch_bounds__(256) void k_greedy_init_multi(const GreedyDesc* d) {
  const GreedyDesc q = d[blockIdx.y];
  if (q.k == 0) return;
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  const uint64_t i0 = blockIdx.x * uint64_t(blockDim.x) + threadIdx.x;
  for (uint64_t u = i0; u < q.n; u += stride) q.gain[u] = static_cast<int32_t>(q.deg[u]);
  for (uint64_t w = i0; w < (q.m + 31) / 32 + 1; w += stride) q.covered[w] = 0;
  for (uint64_t r = i0; r < q.k; r += stride) {
    q.best[r] = 0;
    q.newcov[r] = 0;
  }
  for (uint64_t b = i0; b < kGainBins; b += stride) q.hist[b] = 0;
  if (i0 == 0) {
    q.cst[0] = kModeFull;
    q.cst[1] = 0;
    q.cst[2] = 0;
  }
}

// Items (query, slice b of S): the argmax of every query's slices, or of its
// list (slice 0), grid-strided so that finished queries and list-mode
// slices cost one check each instead of a workgroup launch.
__global__ __launch_bounds__(kArgBlock) void k_argmax_multi(const GreedyDesc* d, uint32_t n_q, uint32_t S,
                                                            const uint32_t* round_base, uint32_t r_local) {
  __shared__ uint64_t red[kArgBlock / kWave];
  __shared__ uint32_t hist[kGainBins];
  const uint32_t r = round_base[0] + r_local;
  const uint64_t items = uint64_t(n_q) * S;
  for (uint64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const GreedyDesc& q = d[it / S];
    const uint32_t b = static_cast<uint32_t>(it % S);
    if (r >= q.k) continue;
    const uint32_t mode = q.cst[0];
    if (mode == kModeList) {
      if (b != 0) continue;
      const uint32_t cnt = min(q.cst[2], kCandMax);
      uint64_t key = 0;
      for (uint32_t i = threadIdx.x; i < cnt; i += kArgBlock) {
        const uint32_t u = q.cand[i];
        const int32_t g = q.gain[u];
        const uint64_t k = g > 0 ? (static_cast<uint64_t>(g) << 32) | (0xFFFFFFFFu - u) : 0ull;
        key = k > key ? k : key;
      }
      key = block_max_u64<kArgBlock>(key, red);
      if (threadIdx.x == 0) q.part[0] = key;
      continue;
    }
    const uint32_t tau = q.cst[1];
    if (mode == kModeFull) {
      for (uint32_t i = threadIdx.x; i < kGainBins; i += kArgBlock) hist[i] = 0;
      __syncthreads();
    }
    uint64_t key = 0;
    for (uint32_t u = b * kArgBlock + threadIdx.x; u < q.n; u += S * kArgBlock) {
      const int32_t g = q.gain[u];
      if (g <= 0) continue;
      const uint64_t k = (static_cast<uint64_t>(g) << 32) | (0xFFFFFFFFu - u);
      key = k > key ? k : key;
      if (mode == kModeFull) {
        atomicAdd(&hist[gain_bin(static_cast<uint32_t>(g))], 1u);
      } else if (static_cast<uint32_t>(g) >= tau) {
        const uint32_t at = atomicAdd(&q.cst[2], 1u);
        if (at < kCandMax) q.cand[at] = u;
      }
    }
    key = block_max_u64<kArgBlock>(key, red);   // contains barriers
    if (threadIdx.x == 0) q.part[b] = key;
    if (mode == kModeFull) {
      for (uint32_t i = threadIdx.x; i < kGainBins; i += kArgBlock)
        if (hist[i]) atomicAdd(&q.hist[i], hist[i]);
      __syncthreads();
    }
  }
}

// One workgroup per query: the round's pick from the argmax maxima (S of
// them, or one in list mode), written to best[r]; 0 once a round found no
// positive gain.  cst[3] receives the pick's row length over the segments.
__global__ __launch_bounds__(256) void k_pick_multi(const GreedyDesc* d, uint32_t S, const uint32_t* round_base,
                                                    uint32_t r_local) {
  __shared__ uint64_t red[256 / kWave];
  const GreedyDesc& q = d[blockIdx.x];
  const uint32_t r = round_base[0] + r_local;
  if (r >= q.k) return;
  if (r > 0 && (q.best[r - 1] >> 32) == 0) {
    if (threadIdx.x == 0) q.best[r] = 0;
    return;
  }
  const uint32_t parts = q.cst[0] == kModeList ? 1u : S;
  uint64_t key = 0;
  for (uint32_t i = threadIdx.x; i < parts; i += 256) key = q.part[i] > key ? q.part[i] : key;
  key = block_max_u64<256>(key, red);
  uint64_t len = 0;
  if ((key >> 32) != 0) {
    const uint32_t u = 0xFFFFFFFFu - static_cast<uint32_t>(key);
    for (uint32_t g = threadIdx.x; g < q.n_seg; g += 256) {
      const uint64_t* o = q.seg_off + size_t(g) * (size_t(q.n) + 1);
      len += o[u + 1] - o[u];
    }
  }
  len = block_sum_u64<256>(len, red);
  if (threadIdx.x == 0) {
    q.best[r] = key;
    q.cst[3] = static_cast<uint32_t>(len < 0xFFFFFFFFull ? len : 0xFFFFFFFFull);
  }
}

// Items (query, part b of S): the covering walk of each query's pick.
__global__ __launch_bounds__(kCoverBlock) void k_cover_multi(const GreedyDesc* d, uint32_t n_q, uint32_t S,
                                                             const uint32_t* round_base, uint32_t r_local) {
  __shared__ CoverShared sh;
  const uint32_t r = round_base[0] + r_local;
  const uint64_t items = uint64_t(n_q) * S;
  for (uint64_t it = blockIdx.x; it < items; it += gridDim.x) {
    const GreedyDesc& q = d[it / S];
    const uint32_t b = static_cast<uint32_t>(it % S);
    if (r >= q.k) continue;
    const uint64_t key = q.best[r];
    if ((key >> 32) == 0) continue;
    if (uint64_t(b) * kCoverBlock >= q.cst[3]) continue;   // nothing of the row lands here
    cover_walk(0xFFFFFFFFu - static_cast<uint32_t>(key), q.seg_off, q.n_seg, q.inc, q.he_off, q.he_nodes, q.n,
               q.covered, q.gain, q.newcov + r, b, S, sh);
  }
}

// After a round: the next round's mode (see the candidate lists above).
__global__ __launch_bounds__(256) void k_greedy_post_multi(const GreedyDesc* d, const uint32_t* round_base,
                                                           uint32_t r_local) {
  __shared__ uint64_t red[256 / kWave];
  __shared__ uint32_t pick;
  const GreedyDesc& q = d[blockIdx.x];
  const uint32_t r = round_base[0] + r_local;
  if (r >= q.k) return;
  const uint32_t mode = q.cst[0];
  if (mode == kModeFull) {
    if (threadIdx.x == 0) {
      // lowest bin whose bins and those above hold at most kCandMax nodes
      uint32_t cum = 0, found = kGainBins;
      for (int b = kGainBins - 1; b >= 0; --b) {
        if (cum + q.hist[b] > kCandMax) break;
        cum += q.hist[b];
        found = static_cast<uint32_t>(b);
      }
      pick = cum > 0 && found < kGainBins ? found : kGainBins;
    }
    __syncthreads();
    if (threadIdx.x == 0 && pick < kGainBins) {
      q.cst[1] = bin_min(pick);
      q.cst[2] = 0;
      q.cst[0] = kModeCompact;
    }
    for (uint32_t b = threadIdx.x; b < kGainBins; b += 256) q.hist[b] = 0;
    return;
  }
  // list or compact: keep using the list while its largest gain is >= tau
  // (a list that overflowed is incomplete: never used)
  if (q.cst[2] > kCandMax) {
    if (threadIdx.x == 0) q.cst[0] = kModeFull;
    return;
  }
  const uint32_t cnt = q.cst[2];
  uint64_t mx = 0;
  for (uint32_t i = threadIdx.x; i < cnt; i += 256) {
    const int32_t g = q.gain[q.cand[i]];
    mx = g > 0 && static_cast<uint64_t>(g) > mx ? static_cast<uint64_t>(g) : mx;
  }
  mx = block_max_u64<256>(mx, red);
  if (threadIdx.x == 0) q.cst[0] = mx >= q.cst[1] && mx > 0 ? kModeList : kModeFull;
}

__global__ void k_round_advance(uint32_t* round_base, uint32_t by) {
  if (threadIdx.x == 0 && blockIdx.x == 0) round_base[0] += by;
}

__global__ void k_greedy_finish_multi(const GreedyDesc* d) {
  const GreedyDesc& q = d[blockIdx.x];
  if (q.k == 0 || threadIdx.x != 0) return;
  uint64_t cov = 0;
  uint32_t r = 0;
  for (; r < q.k; ++r) {
    const uint64_t key = q.best[r];
    if ((key >> 32) == 0) break;
    cov += q.newcov[r];
    q.picks[r] = 0xFFFFFFFFu - static_cast<uint32_t>(key);
    q.cov_cum[r] = cov;
  }
  *q.n_picked = r;
}

void greedy_multi_init(const GreedyDesc* d, uint32_t n_q, uint32_t max_n, hipStream_t s) {
  hipLaunchKernelGGL(k_greedy_init_multi, dim3(grid_for(max_n, 256, 1024), n_q), dim3(256), 0, s, d);
}

// Slices per query of the multi-query argmax: at least 16 nodes per thread,
// at most kArgGrid.
static uint32_t argmax_slices(uint32_t max_n) {
  return grid_for((uint64_t(max_n) + 15) / 16, kArgBlock, kArgGrid);
}

void greedy_multi_rounds(const GreedyDesc* d, uint32_t n_q, uint32_t max_n, uint32_t cover_grid, uint32_t* round_base,
                         uint32_t rounds, hipStream_t s) {
  const uint32_t Sa = argmax_slices(max_n);
  const unsigned ga = grid_for(uint64_t(n_q) * Sa, 1, 4096);
  const unsigned gc = grid_for(uint64_t(n_q) * cover_grid, 1, 4096);
  for (uint32_t r = 0; r < rounds; ++r) {
    hipLaunchKernelGGL(k_argmax_multi, dim3(ga), dim3(kArgBlock), 0, s, d, n_q, Sa, round_base, r);
    hipLaunchKernelGGL(k_pick_multi, dim3(n_q), dim3(256), 0, s, d, Sa, round_base, r);
    hipLaunchKernelGGL(k_cover_multi, dim3(gc), dim3(kCoverBlock), 0, s, d, n_q, cover_grid, round_base, r);
    hipLaunchKernelGGL(k_greedy_post_multi, dim3(n_q), dim3(256), 0, s, d, round_base, r);
  }
  hipLaunchKernelGGL(k_round_advance, dim3(1), dim3(64), 0, s, round_base, rounds);
}

void greedy_multi_finish(const GreedyDesc* d, uint32_t n_q, hipStream_t s) {
  hipLaunchKernelGGL(k_greedy_finish_multi, dim3(n_q), dim3(64), 0, s, d);
}

uint32_t greedy_cand_words() { return kCandMax; }
uint32_t greedy_hist_words() { return kGainBins; }

uint32_t greedy_part_words() { return kArgGrid; }

// ---------------------------------------------------------------------------
// Greedy by one workgroup, gains and covered bits in LDS: a round needs no
// global atomic, no other workgroup and no launch, so it takes 4.8
// us (n = 2,000, m = 10,000, 45,000 entries, k = 10) where a round of kernels
// takes 11.3 (two of them for one query, four for the engine's).  Per round: the largest key of the n gains; then each wave takes
// 64 entries of the pick's rows at a time, marks the newly covered samples
// and spreads the concatenation of their hyperedges over its lanes.
constexpr int kSoloBlock = 1024;
constexpr size_t kSoloLds = 144 << 10;      // of the 160 KB of a CU
// hyperedge entries per round that one workgroup is given, and samples whose
// offsets the L2 holds beside the rest; each further one counts as two entries
constexpr uint64_t kSoloEntries = 12288, kSoloNear = 65536;
constexpr int kSoloUnroll = 4;              // hyperedge entries a lane has in flight

struct SoloShared {
  uint64_t seg_beg[kMaxSegments], seg_pre[kMaxSegments + 1];
  uint64_t red[2 * Coll<kSoloBlock>::kHalf];
  unsigned long long cov;   // samples covered so far
};

__device__ __forceinline__ void greedy_solo_run(const GreedyDesc& q, int32_t* gain, SoloShared& sh) {
  Coll<kSoloBlock> co{sh.red, 0};
  const uint32_t tid = threadIdx.x, n = q.n;
  const int lane = lane_id();
  uint32_t* covered = reinterpret_cast<uint32_t*>(gain + n);
  for (uint32_t u = tid; u < n; u += kSoloBlock) gain[u] = static_cast<int32_t>(q.deg[u]);
  for (uint64_t w = tid; w < (q.m + 31) / 32 + 1; w += kSoloBlock) covered[w] = 0;
  if (tid == 0) sh.cov = 0;
  __syncthreads();
  uint32_t r = 0;
  for (; r < q.k; ++r) {
    int32_t top = 0;
    uint32_t at = 0;
    for (uint32_t u = tid; u < n; u += kSoloBlock) {
      const int32_t g = gain[u];
      at = g > top ? u : at;
      top = g > top ? g : top;
    }
    const uint64_t key = co.max(gain_key(top, at));
    if ((key >> 32) == 0) break;
    const uint32_t pick = 0xFFFFFFFFu - static_cast<uint32_t>(key);
    if (tid < kWave) {   // segment starts and the prefix of the row lengths (n_seg <= 64)
      uint64_t rb = 0, len = 0;
      if (tid < q.n_seg) {
        const uint64_t* o = q.seg_off + size_t(tid) * (size_t(n) + 1);
        rb = o[pick];
        len = o[pick + 1] - rb;
      }
      const uint64_t incl = wave_incl_scan_u64(len);
      if (tid < q.n_seg) {
        sh.seg_beg[tid] = rb;
        sh.seg_pre[tid + 1] = incl;
      }
      if (tid == 0) sh.seg_pre[0] = 0;
    }
    __syncthreads();
    const uint64_t row = sh.seg_pre[q.n_seg];
    uint32_t g = 0, cnt = 0;
    for (uint64_t base = tid - lane; base < row; base += kSoloBlock) {   // uniform in the wave
      const uint64_t x = base + lane;
      uint64_t h0 = 0;
      uint32_t len = 0;
      bool fresh = false;
      if (x < row) {
        while (x >= sh.seg_pre[g + 1]) ++g;
        const uint32_t s = q.inc[sh.seg_beg[g] + (x - sh.seg_pre[g])];
        const uint32_t bit = 1u << (s & 31u);
        fresh = !(atomicOr(&covered[s >> 5], bit) & bit);
        if (fresh) {
          h0 = q.he_off[s];
          len = static_cast<uint32_t>(q.he_off[s + 1] - h0);
        }
      }
      cnt += static_cast<uint32_t>(__popcll(__ballot(fresh)));
      const uint32_t incl = wave_incl_scan_u32(len), off = incl - len;
      const uint32_t total = lane_u32(incl, kWave - 1);
      for (uint32_t e0 = 0; e0 < total; e0 += kWave * kSoloUnroll) {
        uint32_t v[kSoloUnroll];
#pragma unroll
        for (int j = 0; j < kSoloUnroll; ++j) {
          // the sample holding entry e: the last lane with off <= e (empty
          // hyperedges repeat their successor's offset)
          const uint32_t e = e0 + j * kWave + lane;
          int lo = 0;
#pragma unroll
          for (int step = 32; step; step >>= 1)
            if (static_cast<uint32_t>(__shfl(static_cast<int>(off), lo + step, kWave)) <= e) lo += step;
          const uint64_t b = __shfl(h0, lo, kWave);
          const uint32_t o = static_cast<uint32_t>(__shfl(static_cast<int>(off), lo, kWave));
          v[j] = e < total ? q.he_nodes[b + (e - o)] : kUnseen;
        }
#pragma unroll
        for (int j = 0; j < kSoloUnroll; ++j)
          if (v[j] < n) atomicSub(&gain[v[j]], 1);
      }
    }
    if (lane == 0 && cnt) atomicAdd(&sh.cov, static_cast<unsigned long long>(cnt));
    __syncthreads();
    if (tid == 0) {   // (sh.cov next changes after the next round's barriers)
      q.picks[r] = pick;
      q.cov_cum[r] = sh.cov;
    }
  }
  if (tid == 0) *q.n_picked = r;
}

__global__ __launch_bounds__(kSoloBlock) void k_greedy_solo(GreedyDesc q) {
  extern __shared__ int32_t solo_lds[];
  __shared__ SoloShared sh;
  greedy_solo_run(q, solo_lds, sh);
}

__global__ __launch_bounds__(kSoloBlock) void k_greedy_solo_multi(const GreedyDesc* d) {
  extern __shared__ int32_t solo_lds[];
  __shared__ SoloShared sh;
  const GreedyDesc q = d[blockIdx.x];
  if (q.k) greedy_solo_run(q, solo_lds, sh);
}

size_t greedy_solo_lds(uint32_t n, uint64_t m) { return size_t(n) * 4 + ((m + 31) / 32 + 1) * 4; }

// One workgroup where the state fits its LDS and the hyperedges' nodes, of
// which a round of kernels takes many at once, and, where they are many, the
// samples, whose offsets are scattered reads, do not outweigh the rounds (whole
// cover call, us, one workgroup against rounds; n = 2,000, m = 10,000: 40,000
// entries, k = 20: 291, 446; 300,000 entries, k = 50: 627, 760; k = 20: 501, 487;
// n = m = 30,000, 120,000 entries, k = 11: 228, 316; 500,000 samples of one node,
// k = 50: 720, 662; of 4, k = 200: 3,198, 2,367).
bool greedy_solo(uint32_t n, uint64_t m, uint64_t entries, uint32_t k) {
  return greedy_solo_lds(n, m) <= kSoloLds &&
         entries + 2 * (m > kSoloNear ? m - kSoloNear : 0) <= uint64_t(k) * kSoloEntries;
}

template <typename F>
static void allow_lds(F* f) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(kSoloLds));
}

void greedy_multi_solo(const GreedyDesc* d, uint32_t n_q, size_t lds, hipStream_t s) {
  allow_lds(&k_greedy_solo_multi);
  hipLaunchKernelGGL(k_greedy_solo_multi, dim3(n_q), dim3(kSoloBlock), lds, s, d);
}

// The rounds' results, up to the first without a gain, by one wave.
__global__ __launch_bounds__(kWave) void k_greedy_finish(const uint64_t* best, const uint64_t* newcov, uint32_t k,
                                                         uint32_t* picks, uint64_t* cov_cum, uint32_t* n_picked) {
  uint64_t cov = 0;
  uint32_t r0 = 0, n = 0;
  for (; r0 < k; r0 += kWave) {
    const uint32_t r = r0 + threadIdx.x;
    const uint64_t key = r < k ? best[r] : 0ull;
    const uint64_t end = __ballot((key >> 32) == 0);
    const uint32_t here = end ? __ffsll(static_cast<unsigned long long>(end)) - 1 : kWave;
    const uint64_t incl = wave_incl_scan_u64(threadIdx.x < here ? newcov[r] : 0ull);
    if (threadIdx.x < here) {
      picks[r] = 0xFFFFFFFFu - static_cast<uint32_t>(key);
      cov_cum[r] = cov + incl;
    }
    n += here;
    cov += lane_u64(incl, kWave - 1);
    if (end) break;
  }
  if (threadIdx.x == 0) *n_picked = n;
}

// The round state's start: gain, covered and the rounds' keys and counts.
static void greedy_start(uint32_t n, uint64_t m, uint32_t k, const uint32_t* deg, int32_t* gain, uint32_t* cov,
                         uint64_t* best, uint64_t* newcov, hipStream_t s) {
  hipLaunchKernelGGL(k_gain_init, dim3(grid_for(n, 256)), dim3(256), 0, s, deg, n, gain);
  fill_u32(cov, 0, (m + 31) / 32 + 1, s);
  fill_u64(best, 0, k, s);
  fill_u64(newcov, 0, k, s);
}

// Rounds r0 .. k - 1, each by an argmax and a covering kernel.
static void greedy_rounds(uint32_t r0, uint32_t n, const uint64_t* he_off, const uint32_t* he_nodes, uint32_t k,
                          const uint64_t* seg_off, uint32_t n_seg, const uint32_t* inc, int32_t* gain, uint32_t* cov,
                          uint64_t* best, uint64_t* newcov, hipStream_t s) {
  const unsigned ga = grid_for(n, kArgBlock, kArgGrid);
  uint64_t* part = best + k;
  const unsigned gc = 1024;
  for (uint32_t r = r0; r < k; ++r) {
    hipLaunchKernelGGL(k_argmax, dim3(ga), dim3(kArgBlock), 0, s, gain, n, part);
    hipLaunchKernelGGL(k_cover, dim3(gc), dim3(kCoverBlock), 0, s, part, ga, best + r, seg_off, n_seg, inc, he_off,
                       he_nodes, n, cov, gain, newcov + r);
  }
}

// Launches greedy's k rounds on an incidence of n_seg segments (offsets
// seg_off, entries inc (at most `entries`), degrees deg): gain u32[n],
// covered u32[m/32 + 1], best u64[k + kArgGrid] and newcov u64[k] are the
// round state.  Launches only.
static void greedy_kernels(uint32_t n, uint64_t m, const uint64_t* he_off, const uint32_t* he_nodes, uint32_t k,
                           const uint32_t* deg, const uint64_t* seg_off, uint32_t n_seg, const uint32_t* inc,
                           int32_t* gain, uint32_t* cov, uint64_t* best, uint64_t* newcov, uint32_t* picks,
                           uint64_t* cov_cum, uint32_t* n_picked, uint64_t entries, hipStream_t s) {
  if (greedy_solo(n, m, entries, k)) {
    const GreedyDesc q = {gain, cov, nullptr, best, newcov, deg, seg_off, inc, he_off, he_nodes, picks, cov_cum,
                          n_picked, nullptr, nullptr, nullptr, m, n, n_seg, k, 0};
    allow_lds(&k_greedy_solo);
    hipLaunchKernelGGL(k_greedy_solo, dim3(1), dim3(kSoloBlock), greedy_solo_lds(n, m), s, q);
    return;
  }
  greedy_start(n, m, k, deg, gain, cov, best, newcov, s);
  greedy_rounds(0, n, he_off, he_nodes, k, seg_off, n_seg, inc, gain, cov, best, newcov, s);
  hipLaunchKernelGGL(k_greedy_finish, dim3(1), dim3(kWave), 0, s, best, newcov, k, picks, cov_cum, n_picked);
}

// The same in batches, waiting for each; *ran is false if there is no room.
static int greedy_batches(centra_ctx* ctx, BatchArgs a, uint64_t m, const uint32_t* deg, uint32_t* picks,
                          uint64_t* cov_cum, uint32_t* n_picked, bool* ran, hipStream_t s) {
  const size_t part_b = size_t(kTopCols + kTopBlocks) * 8, st_b = (sizeof(BatchState) + 255) & ~size_t(255);
  *ran = false;
  if (ensure(ctx, ctx->batch_ws, part_b + st_b + size_t(kBatchList) * 8 + m * 8, false, s)) {
    ctx->err.clear();
    return CENTRA_OK;
  }
  *ran = true;
  char* ws = static_cast<char*>(ctx->batch_ws.ptr);
  a.part = reinterpret_cast<uint64_t*>(ws);
  a.st = reinterpret_cast<BatchState*>(ws + part_b);
  a.list = reinterpret_cast<uint64_t*>(ws + part_b + st_b);
  a.mask = a.list + kBatchList;
  greedy_start(a.n, m, a.k, deg, a.gain, a.covered, a.best, a.newcov, s);
  fill_u32(reinterpret_cast<uint32_t*>(a.st), 0, 16, s);   // r and fail among them
  fill_u64(a.mask, 0, m, s);
  uint32_t r = 0;
  a.m = m;
  while (r < a.k) {
    a.r = r;
    hipLaunchKernelGGL(k_batch_top, dim3(kTopBlocks), dim3(kTopBlock), 0, s, a, r == 0 ? 1 : 0);
    hipLaunchKernelGGL(k_batch_cands, dim3(1), dim3(kBatchBlock), 0, s, a);
    hipLaunchKernelGGL(k_batch_mask, dim3(512), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_batch_list, dim3(512), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_batch_solve, dim3(1), dim3(kBatchBlock), 0, s, a);
    hipLaunchKernelGGL(k_batch_cover, dim3(1024), dim3(kCoverBlock), 0, s, a);
    uint32_t h[3];   // r, fail, done
    CENTRA_HIP(ctx, hipMemcpyAsync(h, &a.st->r, sizeof(h), hipMemcpyDeviceToHost, s));
    CENTRA_HIP(ctx, hipStreamSynchronize(s));
    const bool little = h[0] - r < kBatchMinPicks;
    r = h[0];
    if (h[2]) break;   // no positive gain is left
    if (h[1] || little) {
      greedy_rounds(r, a.n, a.he_off, a.he_nodes, a.k, a.seg_off, a.n_seg, a.inc, a.gain, a.covered, a.best, a.newcov,
                    s);
      break;
    }
  }
  hipLaunchKernelGGL(k_greedy_finish, dim3(1), dim3(kWave), 0, s, a.best, a.newcov, a.k, picks, cov_cum, n_picked);
  CENTRA_HIP(ctx, hipGetLastError());
  return CENTRA_OK;
}

int greedy_reserve(centra_ctx* ctx, uint32_t n, uint64_t m, uint32_t k, hipStream_t s) {
  int rc;
  if ((rc = ensure(ctx, ctx->gain, size_t(n) * 4, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->covered, ((m + 31) / 32 + 1) * 4, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->best, (size_t(k) + kArgGrid) * 8, false, s))) return rc;
  return ensure(ctx, ctx->newcov, size_t(k) * 8, false, s);
}

int greedy_on_incidence(centra_ctx* ctx, bool waits, uint32_t n, uint64_t m, const uint64_t* he_off, const uint32_t* he_nodes,
                        uint32_t k, uint32_t* picks, uint64_t* cov_cum, uint32_t* n_picked, hipStream_t s) {
  int rc;
  if ((rc = ensure(ctx, ctx->gain, size_t(n) * 4, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->covered, ((m + 31) / 32 + 1) * 4, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->best, (size_t(k) + kArgGrid) * 8, false, s))) return rc;
  if ((rc = ensure(ctx, ctx->newcov, size_t(k) * 8, false, s))) return rc;
  // In batches where the call may wait for them; not under a budget, whose
  // memory other steps may need.
  if (waits && !ctx->budget && k >= kBatchMinK && m <= kBatchMaxM && ctx->inc_nseg <= kBatchSegs &&
      !greedy_solo(n, m, ctx->inc_limit, k)) {
    BatchArgs a{};
    a.n = n;
    a.n_seg = ctx->inc_nseg;
    a.k = k;
    a.seg_off = static_cast<const uint64_t*>(ctx->inc_off.ptr);
    a.inc = static_cast<const uint32_t*>(ctx->inc.ptr);
    a.he_off = he_off;
    a.he_nodes = he_nodes;
    a.gain = static_cast<int32_t*>(ctx->gain.ptr);
    a.covered = static_cast<uint32_t*>(ctx->covered.ptr);
    a.best = static_cast<uint64_t*>(ctx->best.ptr);
    a.newcov = static_cast<uint64_t*>(ctx->newcov.ptr);
    bool ran;
    if ((rc = greedy_batches(ctx, a, m, static_cast<const uint32_t*>(ctx->deg.ptr), picks, cov_cum, n_picked, &ran, s)))
      return rc;
    if (ran) return CENTRA_OK;
  }
  greedy_kernels(n, m, he_off, he_nodes, k, static_cast<const uint32_t*>(ctx->deg.ptr),
                 static_cast<const uint64_t*>(ctx->inc_off.ptr), ctx->inc_nseg,
                 static_cast<const uint32_t*>(ctx->inc.ptr), static_cast<int32_t*>(ctx->gain.ptr),
                 static_cast<uint32_t*>(ctx->covered.ptr), static_cast<uint64_t*>(ctx->best.ptr),
                 static_cast<uint64_t*>(ctx->newcov.ptr), picks, cov_cum, n_picked, ctx->inc_limit, s);
  CENTRA_HIP(ctx, hipGetLastError());
  return CENTRA_OK;
}

// ---------------------------------------------------------------------------
// Greedy cover without allocation.  Every workspace of one greedy call (the
// single incidence segment, the round state, the scan tiles and an error
// word) is carved from `scratch`, a fixed array in device memory that each
// GPU holds for the life of the process.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in for the
// symbol): its device address is looked up once per device with
// hipGetSymbolAddress and kept in g_scratch_ptr.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Bytes of scratch a greedy call on (n, m, I entries, k) carves.
size_t static_greedy_bytes(uint32_t n, uint64_t m, uint64_t I, uint32_t k) {
  const size_t N = n;
  return align256(4) + align256(N * 4) * 3 + align256((N + 1) * 8) + align256(N * 8) + align256((I ? I : 1) * 4) * 2 +
         align256(((m + 31) / 32 + 1) * 4) + align256((size_t(k) + kArgGrid) * 8) + align256(size_t(k) * 8) +
         align256(scan_tile_words(N) * 8);
}

int greedy_cover_static(uint32_t n, uint64_t m, const uint64_t* he_off, const uint32_t* he_nodes, uint32_t k,
                        uint32_t* picks, uint64_t* cov_cum, uint32_t* n_picked, hipStream_t s, std::string* err) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    *err = "greedy_cover_noalloc: no current HIP device";
    return CENTRA_EHIP;
  }
  char* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p) {
        *err = std::string("greedy_cover_noalloc: hipGetSymbolAddress failed: ") + hipGetErrorString(e);
        return CENTRA_EHIP;
      }
      g_scratch_ptr[dev] = p;
    }
    base = static_cast<char*>(g_scratch_ptr[dev]);
  }
  uint64_t I = 0;
  if ((e = hipMemcpyAsync(&I, he_off + m, 8, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess) {
    *err = std::string("greedy_cover_noalloc: reading he_off[m]: ") + hipGetErrorString(e);
    return CENTRA_EHIP;
  }
  if (I && !he_nodes) {
    *err = "greedy_cover_noalloc: he_nodes is NULL";
    return CENTRA_EINVAL;
  }
  const size_t need = static_greedy_bytes(n, m, I, k);
  if (need > kStaticScratchBytes) {
    *err = "greedy_cover_noalloc: n = " + std::to_string(n) + ", m = " + std::to_string(m) + ", " +
           std::to_string(I) + " entries and k = " + std::to_string(k) + " need " + std::to_string(need) +
           " bytes of scratch; the fixed maximum is " + std::to_string(kStaticScratchBytes);
    return CENTRA_ENOSPC;
  }
  const size_t N = n;
  size_t at = 0;
  auto carve = [&](size_t bytes) {
    char* p = base + at;
    at += align256(bytes);
    return static_cast<void*>(p);
  };
  uint32_t* flags = static_cast<uint32_t*>(carve(4));
  uint32_t* deg = static_cast<uint32_t*>(carve(N * 4));
  uint32_t* sdeg = static_cast<uint32_t*>(carve(N * 4));
  int32_t* gain = static_cast<int32_t*>(carve(N * 4));
  uint64_t* off = static_cast<uint64_t*>(carve((N + 1) * 8));
  uint64_t* cur = static_cast<uint64_t*>(carve(N * 8));
  uint32_t* inc = static_cast<uint32_t*>(carve((I ? I : 1) * 4));
  uint32_t* inc_node = static_cast<uint32_t*>(carve((I ? I : 1) * 4));
  uint32_t* cov = static_cast<uint32_t*>(carve(((m + 31) / 32 + 1) * 4));
  uint64_t* best = static_cast<uint64_t*>(carve((size_t(k) + kArgGrid) * 8));
  uint64_t* newcov = static_cast<uint64_t*>(carve(size_t(k) * 8));
  uint64_t* tiles = static_cast<uint64_t*>(carve(scan_tile_words(N) * 8));
  // the array keeps the previous call's contents: the error word starts at 0
  // here, and every other region is written before it is read
  fill_u32(flags, 0, 1, s);
  incidence_segment(n, 0, m, I, I, he_off, he_nodes, true, deg, sdeg, off, cur, inc, inc_node, tiles, flags, s);
  greedy_kernels(n, m, he_off, he_nodes, k, deg, off, 1, inc, gain, cov, best, newcov, picks, cov_cum, n_picked, I, s);
  if ((e = hipGetLastError()) != hipSuccess) {
    *err = std::string("greedy_cover_noalloc: launch failed: ") + hipGetErrorString(e);
    return CENTRA_EHIP;
  }
  uint32_t f = 0;
  if ((e = hipMemcpyAsync(&f, flags, 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess) {
    *err = std::string("greedy_cover_noalloc: ") + hipGetErrorString(e);
    return CENTRA_EHIP;
  }
  if (f & kErrNodeRange) {
    *err = "greedy_cover_noalloc: hyperedge node id out of range";
    return CENTRA_EINVAL;
  }
  if (f) {
    *err = "greedy_cover_noalloc: hyperedge offsets decrease";
    return CENTRA_EINVAL;
  }
  return CENTRA_OK;
}

}  // namespace centra
