// AMCERA ingredients on gfx950: Rademacher sign words, the per-node trial
// sums R[u][j] = sum_{s : u in h_s} sigma_js, the per-trial sums of the k
// largest positive R[.][j], the k largest deg_H(u) and max |h|.
//
// Signs.  Sample s gets Wt = ceil(t/64) words; word w holds trials
// 64w .. 64w+63 and is word (w mod 4) of Philox block (w div 4, s,
// instance, 1), so bit (j mod 64) of word j div 64 is sigma_js.
//
// Trial sums.  R[u][j] = 2 P[u][j] - deg_H(u) with P[u][j] the number of
// samples of u's incidence row whose bit j is set.  A wave walks a span of
// the incidence (grouped by node), lane j counting trial j (k_rade_count).
//
// Top-k.  The t columns of R and the column of degrees are selected over the
// node-major P itself (columns_topk), or, for the engine, which keeps R by
// trial, over rows (select_topk_rows): for every row the k-th largest
// positive value is found by MSD radix selection: a histogram over the bit
// length, then 10-bit digit histograms below the leading bit, each with
// per-bin counts and sums; the answer is the sum of every value above the
// selected one plus the remaining copies of it.  Each pass splits every row
// over many workgroups, which build LDS histograms and merge them into the
// row's global histogram with atomics (a row on one workgroup would leave
// most CUs idle and serialise on a few LDS bins); a one-wave kernel per row
// then picks the digit with a wave scan and clears the histogram.
#include <algorithm>
#include <vector>

#include "common.hpp"
#include "internal.hpp"

namespace centra {

__global__ void k_rade_words(uint64_t seed, uint32_t instance, uint64_t s0, uint64_t s1, uint32_t Wt,
                             uint64_t* words) {
  const uint32_t nblk = (Wt + 3) / 4;
  const uint64_t total = (s1 - s0) * nblk;
  for (uint64_t x = blockIdx.x * uint64_t(blockDim.x) + threadIdx.x; x < total;
       x += uint64_t(gridDim.x) * blockDim.x) {
    const uint64_t s = s0 + x / nblk;
    const uint32_t b = static_cast<uint32_t>(x % nblk);
    const Block4 r = philox4x64_10(b, s, instance, 1, seed, 0);
    uint64_t* dst = words + s * Wt + 4ull * b;
    const uint32_t avail = Wt - 4 * b;
    dst[0] = r.w0;
    if (avail > 1) dst[1] = r.w1;
    if (avail > 2) dst[2] = r.w2;
    if (avail > 3) dst[3] = r.w3;
  }
}

static unsigned grid_for(uint64_t n, unsigned block, unsigned cap = 16384) {
  uint64_t g = (n + block - 1) / block;
  if (g > cap) g = cap;
  return g ? static_cast<unsigned>(g) : 1u;
}

int rade_words(centra_ctx* ctx, uint64_t seed, uint32_t instance, uint64_t s0, uint64_t s1, uint32_t t,
               hipStream_t s) {
  const uint32_t Wt = (t + 63) / 64;
  ctx->mc_ok = false;   // the extend calls' AMCERA state is valid only after their own updates
  ++ctx->words_gen;
  int rc = ensure(ctx, ctx->words, size_t(s1) * Wt * 8, true, s);
  if (rc) return rc;
  if (s1 > s0)
    hipLaunchKernelGGL(k_rade_words, dim3(grid_for((s1 - s0) * ((Wt + 3) / 4), 256)), dim3(256), 0, s, seed,
                       instance, s0, s1, Wt, static_cast<uint64_t*>(ctx->words.ptr));
  CENTRA_HIP(ctx, hipGetLastError());
  return CENTRA_OK;
}

// ---------------------------------------------------------------------------
constexpr int kCountBlock = 256;
constexpr uint32_t kCountWaves = 16384;   // two fills of the device

// P[u][j] += number of samples in u's incidence row whose sign bit j is set,
// for the trials 64g .. 64g+63 of word group g = blockIdx.y.  The entries are
// cut into equal spans of whole 64-entry batches, one per wave of the grid
// (a node's entries are consecutive); a wave walks its span one entry at a
// time: the entry's node and sign word are read into scalar registers
// (readlane) and lane j adds bit j of the word to its running count, flushed
// when the node changes.  The cost per entry is a few instructions whatever
// the row lengths; loads are 64 entries per batch, coalesced for the
// incidence, one 8-byte gather per entry for the word, and are under way one
// (words) or two (incidence) batches ahead.  What bounds a short sample is
// the length of the spans, so they are as short as the grid allows: fixed
// spans of 1,024 entries took 92 us from 10,000 samples (45,000 entries), ten
// trials, where this takes 7.6.
//
// A run of entries that both starts and ends inside the span is the node's
// whole row of its segment: with `whole` (the range is one segment and P is
// zero, so a node has no other run) its counts are stored, the others are
// added atomically (spans may split a row).  (Atomics execute in memory on this card: n = 10^6, 4.5M entries, 64
// trials, 191 us with atomics alone, 114 with stores.)
__global__ __launch_bounds__(kCountBlock) void k_rade_count(const uint32_t* inc, const uint32_t* inc_node,
                                                            const uint64_t* he_off, uint64_t m0, uint64_t m1,
                                                            uint64_t limit, const uint64_t* words, uint32_t Wt,
                                                            uint32_t t, int whole, int32_t* P) {
  const int lane = lane_id();
  const uint32_t g = blockIdx.y;
  // the segment's entries [he_off[m0], he_off[m1]) of inc, read on the device
  const uint64_t I0 = he_off[m0], I = he_off[m1];
  if (I > limit || I0 > I) return;   // beyond the incidence (the build raised the error)
  const uint64_t waves = uint64_t(gridDim.x) * (kCountBlock / kWave);
  const uint64_t span = (((I - I0 + waves - 1) / waves + kWave - 1) / kWave) * kWave;
  const uint64_t wave = (blockIdx.x * uint64_t(kCountBlock) + uniform_u32(threadIdx.x)) / kWave;
  const uint64_t e0 = I0 + wave * span;
  if (e0 >= I) return;
  const uint64_t e1 = e0 + span < I ? e0 + span : I;
  const uint32_t jt = 64 * g + lane;   // this lane's trial
  const bool live = jt < t;
  const uint32_t shift = lane & 31;
  const bool high = lane >= 32;
  uint32_t cur = kUnseen;
  uint32_t acc = 0;
  bool open = true;   // the run may have begun before the span
  auto node_of = [&](uint64_t e) { return e < e1 ? inc_node[e] : kUnseen; };
  auto word_of = [&](uint64_t e, uint32_t s) { return e < e1 ? words[uint64_t(s) * Wt + g] : 0ull; };
  uint32_t u = node_of(e0 + lane), u1 = node_of(e0 + kWave + lane);
  uint64_t word = word_of(e0 + lane, e0 + lane < e1 ? inc[e0 + lane] : 0u);
  uint32_t s1 = e0 + kWave + lane < e1 ? inc[e0 + kWave + lane] : 0u;
  for (uint64_t base = e0; base < e1; base += kWave) {
    const uint64_t far = base + 2 * kWave + lane;
    const uint64_t word1 = word_of(base + kWave + lane, s1);
    const uint32_t u2 = node_of(far);
    s1 = far < e1 ? inc[far] : 0u;
    const uint32_t wlo = static_cast<uint32_t>(word), whi = static_cast<uint32_t>(word >> 32);
    const uint32_t cnt = e1 - base < kWave ? static_cast<uint32_t>(e1 - base) : kWave;
    for (uint32_t i = 0; i < cnt; ++i) {
      const uint32_t ui = lane_u32(u, i), lo = lane_u32(wlo, i), hi = lane_u32(whi, i);
      if (ui != cur) {
        if (cur != kUnseen && live) {
          int32_t* p = &P[uint64_t(cur) * t + jt];
          if (whole && !open)
            *p = static_cast<int32_t>(acc);
          else if (acc)
            atomicAdd(p, static_cast<int32_t>(acc));
        }
        open = cur == kUnseen;
        cur = ui;
        acc = 0;
      }
      acc += ((high ? hi : lo) >> shift) & 1u;
    }
    u = u1;
    u1 = u2;
    word = word1;
  }
  if (live && acc) atomicAdd(&P[uint64_t(cur) * t + jt], static_cast<int32_t>(acc));
}

// R[u][j] = 2 P[u][j] - deg[u].
__global__ void k_rade_rows(const int32_t* P, const uint32_t* deg, uint32_t n, uint32_t t, int32_t* R) {
  const uint64_t total = uint64_t(n) * t;
  for (uint64_t i = blockIdx.x * uint64_t(blockDim.x) + threadIdx.x; i < total; i += uint64_t(gridDim.x) * blockDim.x)
    R[i] = 2 * P[i] - static_cast<int32_t>(deg[i / t]);
}

// R[j][u] = 2 P[u][j] - deg[u] (trial-major, for the selection over rows).
// 64 x 64 tiles through LDS.
__global__ __launch_bounds__(256) void k_rade_finish(const int32_t* P, const uint32_t* deg, uint32_t n, uint32_t t,
                                                     int32_t* Rtm) {
  __shared__ int32_t tile[64][65];
  const uint32_t u0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;   // 64 x 4
  for (int r = ty; r < 64; r += 4) {
    const uint32_t u = u0 + r, j = j0 + tx;
    int32_t v = 0;
    if (u < n && j < t) v = 2 * P[uint64_t(u) * t + j] - static_cast<int32_t>(deg[u]);
    tile[r][tx] = v;
  }
  __syncthreads();
  for (int r = ty; r < 64; r += 4) {
    const uint32_t j = j0 + r, u = u0 + tx;
    if (u < n && j < t) Rtm[uint64_t(j) * n + u] = tile[tx][r];
  }
}

// ---------------------------------------------------------------------------
constexpr int kSelBlock = 256;
constexpr int kDigitBits = 10;
constexpr uint32_t kBins = 1u << kDigitBits;   // also holds the 32 bit-length bins
constexpr int kDigitPasses = (30 + kDigitBits - 1) / kDigitBits;   // bits below the leading one

// Selection state of one row: the values still sought have bit length blen
// and their top pbits bits equal prefix; need of them are still to be taken
// and acc holds the sum of the values already taken.
// When done, the row's k largest are its values above tau and `ties`
// copies of tau (tau = 0, ties = 0: all of its positive values, fewer than
// k).
struct SelState {
  uint32_t prefix, pbits, blen, need, done, ties;
  int64_t acc;
  uint32_t tau, pad;
};

__global__ void k_sel_init(SelState* st, const SelRow* rows, uint32_t n_rows, uint32_t* hcnt, uint64_t* hsum) {
  const uint64_t nb = uint64_t(n_rows) * kBins;
  for (uint64_t i = blockIdx.x * uint64_t(blockDim.x) + threadIdx.x; i < nb; i += uint64_t(gridDim.x) * blockDim.x) {
    hcnt[i] = 0;
    hsum[i] = 0;
    if (i < n_rows) {
      const uint32_t k = rows[i].k;
      st[i] = SelState{1, 1, 0, k, k == 0 ? 1u : 0u, 0, 0, 0, 0};
    }
  }
}

// Pass `first`: bit lengths (bins 1..31) of the positive values; else the
// next digit of the values matching the row's prefix.  Block (x, r) takes
// values [x chunk, (x+1) chunk) of row r, chunk = ceil(n_r / gridDim.x).
__global__ __launch_bounds__(kSelBlock) void k_sel_hist(const SelRow* rows, const SelState* st, int first,
                                                        uint32_t* hcnt, uint64_t* hsum) {
  __shared__ uint32_t cnt[kBins];
  __shared__ uint64_t sum[kBins];
  const uint32_t r = blockIdx.y;
  const SelState s = st[r];
  if (s.done) return;
  const SelRow d = rows[r];
  const uint64_t chunk = (uint64_t(d.n) + gridDim.x - 1) / gridDim.x;
  const uint64_t i0 = uint64_t(blockIdx.x) * chunk;
  if (i0 >= d.n) return;
  const uint32_t B = s.blen, up = B - s.pbits;
  const uint32_t nb = first ? 5u : (up < uint32_t(kDigitBits) ? up : uint32_t(kDigitBits));
  const uint32_t shift = first ? 0u : up - nb;
  const uint32_t nbins = first ? 32u : 1u << nb;
  for (uint32_t b = threadIdx.x; b < nbins; b += kSelBlock) {
    cnt[b] = 0;
    sum[b] = 0;
  }
  __syncthreads();
  const int32_t* row = d.vals;
  const uint64_t i1 = i0 + chunk < d.n ? i0 + chunk : d.n;
  for (uint64_t i = i0 + threadIdx.x; i < i1; i += kSelBlock) {
    const int32_t x = row[i];
    if (x <= 0) continue;
    const uint32_t ux = static_cast<uint32_t>(x);
    uint32_t bin;
    if (first) {
      bin = bitlen32(ux);
    } else {
      if ((ux >> up) != s.prefix) continue;
      bin = (ux >> shift) & (nbins - 1u);
    }
    atomicAdd(&cnt[bin], 1u);
    atomicAdd(reinterpret_cast<unsigned long long*>(&sum[bin]), static_cast<unsigned long long>(ux));
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < nbins; b += kSelBlock) {
    if (cnt[b]) {
      atomicAdd(&hcnt[uint64_t(r) * kBins + b], cnt[b]);
      atomicAdd(reinterpret_cast<unsigned long long*>(&hsum[uint64_t(r) * kBins + b]),
                static_cast<unsigned long long>(sum[b]));
    }
  }
}

// One wave per row: walking the bins from the top, the bin where the count
// reaches `need` is the next digit (or bit length); the bins above it are
// taken whole.  Clears the row's histogram for the next pass.
__global__ __launch_bounds__(kWave) void k_sel_decide(SelState* st, int first, uint32_t* hcnt, uint64_t* hsum) {
  const uint32_t r = blockIdx.x;
  const int lane = lane_id();
  SelState s = st[r];
  if (s.done) return;
  const uint32_t up = s.blen - s.pbits;
  const uint32_t nb = first ? 5u : (up < uint32_t(kDigitBits) ? up : uint32_t(kDigitBits));
  const uint32_t nbins = first ? 32u : 1u << nb;
  const uint32_t per = nbins > uint32_t(kWave) ? nbins / kWave : 1u;
  uint32_t* C = hcnt + uint64_t(r) * kBins;
  uint64_t* S = hsum + uint64_t(r) * kBins;
  // lane L owns bins [hi - per, hi) with hi = nbins - L per (top bins first)
  const bool owns = uint32_t(lane) * per < nbins;
  const uint32_t hi = owns ? nbins - uint32_t(lane) * per : 0u;
  uint32_t c = 0;
  uint64_t sm = 0;
  for (uint32_t b = hi; b > hi - (owns ? per : 0u); --b) {
    c += C[b - 1];
    sm += S[b - 1];
  }
  const uint32_t c_incl = wave_incl_scan_u32(c);
  const uint64_t s_incl = wave_incl_scan_u64(sm);
  const uint32_t c_excl = c_incl - c;
  const uint64_t f = __ballot(owns && c_excl < s.need && c_incl >= s.need);
  if (f == 0) {
    // fewer than `need` values left (only in the first pass: fewer than k
    // positive values): all of them are taken
    if (lane == kWave - 1) {
      s.acc += static_cast<int64_t>(s_incl);
      s.done = 1;
      s.tau = 0;
      s.ties = 0;
      st[r] = s;
    }
  } else if (lane == __ffsll(static_cast<unsigned long long>(f)) - 1) {
    uint32_t rem = s.need - c_excl;
    int64_t acc = s.acc + static_cast<int64_t>(s_incl - sm);
    uint32_t d = hi - 1;
    for (uint32_t b = hi; b > hi - per; --b) {
      d = b - 1;
      if (C[d] < rem) {
        rem -= C[d];
        acc += static_cast<int64_t>(S[d]);
      } else {
        break;
      }
    }
    if (first) {
      s.blen = d;
      s.prefix = 1;
      s.pbits = 1;
    } else {
      s.prefix = (s.prefix << nb) | d;
      s.pbits += nb;
    }
    s.need = rem;
    s.acc = acc;
    if (s.pbits >= s.blen) {   // every bit fixed: the remaining copies of prefix
      s.acc += static_cast<int64_t>(s.need) * static_cast<int64_t>(s.prefix);
      s.tau = s.prefix;
      s.ties = s.need;
      s.done = 1;
    }
    st[r] = s;
  }
  for (uint32_t b = lane; b < nbins; b += kWave) {
    C[b] = 0;
    S[b] = 0;
  }
}

// b_max = max(b_max, largest |h| of samples [0, m) of he_off): one atomic
// per workgroup (an atomic per wave on the one word serialised the kernel).
constexpr int kBmaxBlock = 256;
__global__ __launch_bounds__(kBmaxBlock) void k_bmax(const uint64_t* he_off, uint64_t m, uint32_t* b_max) {
  __shared__ uint32_t red[kBmaxBlock / kWave];
  uint32_t mx = 0;
  for (uint64_t s = blockIdx.x * uint64_t(kBmaxBlock) + threadIdx.x; s < m; s += uint64_t(gridDim.x) * kBmaxBlock) {
    const uint64_t len = he_off[s + 1] - he_off[s];
    mx = len > mx ? static_cast<uint32_t>(len) : mx;
  }
  for (int o = 32; o >= 1; o >>= 1) {
    const uint32_t x = __shfl_xor(mx, o, kWave);
    mx = x > mx ? x : mx;
  }
  if (lane_id() == 0) red[threadIdx.x / kWave] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = 0;
    for (int i = 0; i < kBmaxBlock / kWave; ++i) r = red[i] > r ? red[i] : r;
    if (r) atomicMax(b_max, r);
  }
}

__global__ void k_sel_out(const SelState* st, const SelRow* rows, uint32_t n_rows) {
  for (uint32_t r = blockIdx.x * blockDim.x + threadIdx.x; r < n_rows; r += gridDim.x * blockDim.x)
    if (rows[r].out) *rows[r].out = st[r].acc;
}

size_t select_ws_bytes(uint32_t n_rows) { return size_t(n_rows) * (sizeof(SelState) + kBins * 12); }

// The sum of the k largest positive values of every row (rows[r].k, 0 if
// there are none; rows[r].out receives it): MSD radix selection, each pass
// spread over about 2,048 workgroups.
void select_topk_rows(const SelRow* rows, uint32_t n_rows, uint32_t max_n, void* ws, hipStream_t s) {
  SelState* st = static_cast<SelState*>(ws);
  uint64_t* hsum = reinterpret_cast<uint64_t*>(st + n_rows);
  uint32_t* hcnt = reinterpret_cast<uint32_t*>(hsum + size_t(n_rows) * kBins);
  // about 2,048 workgroups per histogram pass, at least 4,096 values each
  uint32_t parts = 2048 / n_rows ? 2048 / n_rows : 1u;
  const uint32_t max_parts = (max_n + 4095) / 4096 ? (max_n + 4095) / 4096 : 1u;
  if (parts > max_parts) parts = max_parts;
  hipLaunchKernelGGL(k_sel_init, dim3(grid_for(uint64_t(n_rows) * kBins, 256)), dim3(256), 0, s, st, rows, n_rows, hcnt,
                     hsum);
  for (int pass = 0; pass <= kDigitPasses; ++pass) {
    hipLaunchKernelGGL(k_sel_hist, dim3(parts, n_rows), dim3(kSelBlock), 0, s, rows, st, pass == 0 ? 1 : 0, hcnt, hsum);
    hipLaunchKernelGGL(k_sel_decide, dim3(n_rows), dim3(kWave), 0, s, st, pass == 0 ? 1 : 0, hcnt, hsum);
  }
  hipLaunchKernelGGL(k_sel_out, dim3(grid_for(n_rows, 256, 64)), dim3(256), 0, s, st, rows, n_rows);
}

// Top-k sums of every row for every k <= K at once: after the selection
// at K, the row's values above its threshold are gathered (at most K of
// them), sorted in LDS together with the threshold's copies, and
// prefix-summed: out[r * K + i] = the sum of the i + 1 largest positive
// values (flat once they run out).
constexpr uint32_t kPrefixMax = 2048;

__global__ __launch_bounds__(kSelBlock) void k_sel_gather(const SelRow* rows, const SelState* st, uint32_t K,
                                                          uint32_t* gcount, int32_t* buf) {
  const uint32_t r = blockIdx.y;
  const SelRow d = rows[r];
  const uint32_t tau = st[r].tau;
  const uint64_t chunk = (uint64_t(d.n) + gridDim.x - 1) / gridDim.x;
  const uint64_t i0 = uint64_t(blockIdx.x) * chunk;
  const uint64_t i1 = i0 + chunk < d.n ? i0 + chunk : d.n;
  for (uint64_t i = i0 + threadIdx.x; i < i1; i += kSelBlock) {
    const int32_t x = d.vals[i];
    if (x <= 0 || static_cast<uint32_t>(x) <= tau) continue;
    const uint32_t at = atomicAdd(&gcount[r], 1u);
    if (at < K) buf[size_t(r) * K + at] = x;
  }
}

__global__ __launch_bounds__(kSelBlock) void k_sel_prefix(const SelState* st, const uint32_t* gcount,
                                                          const int32_t* buf, uint32_t K, uint32_t Kpad,
                                                          int64_t* out) {
  __shared__ int32_t v[kPrefixMax];
  __shared__ int64_t wsum[kSelBlock / kWave];
  const uint32_t r = blockIdx.x;
  const SelState s = st[r];
  const uint32_t g = gcount[r] < K ? gcount[r] : K;
  for (uint32_t i = threadIdx.x; i < Kpad; i += kSelBlock) {
    int32_t x = 0;
    if (i < g)
      x = buf[size_t(r) * K + i];
    else if (i < g + s.ties && i < K)
      x = static_cast<int32_t>(s.tau);
    v[i] = x;
  }
  __syncthreads();
  // bitonic sort, descending
  for (uint32_t size = 2; size <= Kpad; size <<= 1) {
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (uint32_t i = threadIdx.x; i < Kpad; i += kSelBlock) {
        const uint32_t j = i ^ stride;
        if (j > i) {
          const bool desc = (i & size) == 0;
          const int32_t a = v[i], b = v[j];
          if (desc ? a < b : a > b) {
            v[i] = b;
            v[j] = a;
          }
        }
      }
      __syncthreads();
    }
  }
  // prefix sums: each thread sums Kpad / kSelBlock consecutive entries
  const uint32_t per = Kpad / kSelBlock ? Kpad / kSelBlock : 1u;
  const uint32_t b0 = threadIdx.x * per;
  int64_t loc = 0;
  for (uint32_t i = b0; i < b0 + per && i < Kpad; ++i) loc += v[i];
  const int64_t incl = static_cast<int64_t>(wave_incl_scan_u64(static_cast<uint64_t>(loc)));
  if (lane_id() == kWave - 1) wsum[threadIdx.x / kWave] = incl;
  __syncthreads();
  int64_t run = incl - loc;
  for (uint32_t w = 0; w < threadIdx.x / kWave; ++w) run += wsum[w];
  for (uint32_t i = b0; i < b0 + per && i < Kpad; ++i) {
    run += v[i];
    if (i < K) out[size_t(r) * K + i] = run;
  }
}

size_t select_prefix_ws_bytes(uint32_t n_rows, uint32_t K) {
  return select_ws_bytes(n_rows) + size_t(n_rows) * 4 + size_t(n_rows) * K * 4 + 256;
}

void select_prefix_rows(const SelRow* rows, uint32_t n_rows, uint32_t max_n, uint32_t K, void* ws, int64_t* out,
                        hipStream_t s) {
  select_topk_rows(rows, n_rows, max_n, ws, s);
  const SelState* st = static_cast<const SelState*>(ws);
  uint32_t* gcount = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + select_ws_bytes(n_rows));
  int32_t* buf = reinterpret_cast<int32_t*>(gcount + n_rows);
  fill_u32(gcount, 0, n_rows, s);
  uint32_t parts = 2048 / n_rows ? 2048 / n_rows : 1u;
  const uint32_t max_parts = (max_n + 4095) / 4096 ? (max_n + 4095) / 4096 : 1u;
  if (parts > max_parts) parts = max_parts;
  hipLaunchKernelGGL(k_sel_gather, dim3(parts, n_rows), dim3(kSelBlock), 0, s, rows, st, K, gcount, buf);
  uint32_t Kpad = kSelBlock;
  while (Kpad < K) Kpad <<= 1;
  hipLaunchKernelGGL(k_sel_prefix, dim3(n_rows), dim3(kSelBlock), 0, s, st, static_cast<const uint32_t*>(gcount),
                     static_cast<const int32_t*>(buf), K, Kpad, out);
}

// Launch-only steps of the AMCERA for callers that own their buffers.
void rade_words_launch(uint64_t seed, uint32_t instance, uint64_t s0, uint64_t s1, uint32_t t, uint64_t* words,
                       hipStream_t s) {
  const uint32_t Wt = (t + 63) / 64;
  if (s1 > s0)
    hipLaunchKernelGGL(k_rade_words, dim3(grid_for((s1 - s0) * ((Wt + 3) / 4), 256)), dim3(256), 0, s, seed, instance,
                       s0, s1, Wt, words);
}

void rade_count_launch(const uint32_t* inc, const uint32_t* inc_node, const uint64_t* he_off, uint64_t m0, uint64_t m1,
                       uint64_t span_cap, uint64_t limit, const uint64_t* words, uint32_t t, bool whole, int32_t* P,
                       hipStream_t s) {
  const uint32_t Wt = (t + 63) / 64;
  if (m1 > m0 && span_cap) {
    uint64_t waves = (span_cap + kWave - 1) / kWave;
    if (waves > kCountWaves) waves = kCountWaves;
    const uint64_t blocks = (waves * kWave + kCountBlock - 1) / kCountBlock;
    hipLaunchKernelGGL(k_rade_count, dim3(static_cast<unsigned>(blocks), Wt), dim3(kCountBlock), 0, s, inc, inc_node,
                       he_off, m0, m1, limit, words, Wt, t, whole ? 1 : 0, P);
  }
}

void rade_finish_launch(const int32_t* P, const uint32_t* deg, uint32_t n, uint32_t t, int32_t* Rtm, hipStream_t s) {
  hipLaunchKernelGGL(k_rade_finish, dim3((n + 63) / 64, (t + 63) / 64), dim3(256), 0, s, P, deg, n, t, Rtm);
}

void bmax_launch(const uint64_t* he_off, uint64_t m0, uint64_t m1, uint32_t* b_max, hipStream_t s) {
  if (m1 > m0)
    hipLaunchKernelGGL(k_bmax, dim3(grid_for(m1 - m0, kBmaxBlock, 512)), dim3(kBmaxBlock), 0, s, he_off + m0, m1 - m0,
                       b_max);
}

// ---------------------------------------------------------------------------
// Sums of the k largest positive values of the t columns of R = 2 P - deg and
// of the column of degrees, without R: a lane reads its trial's column of the
// node-major P.  The k-th largest value of a column is narrowed down to a
// range [lo, lo + 2^w): first by bins of 8 to the octave (values below 16 have
// bins of their own), then by 256 bins of the range a pass, then the values
// above it are summed.  R[u][j] <= deg[u], so a pass reads only the rows of
// nodes whose degree reaches some open range of its 64 trials: mostly the
// first pass is the only one over all of P, and it is bound by reading it.
// Each workgroup has its own counts in LDS and writes them out; a workgroup
// per column adds them up.  n = 10^6, t = 64 (k = 50): 377 us with R written by
// trial and selected by rows, 215 so.
constexpr int kColBlock = 1024;
constexpr uint32_t kColParts = 256;   // workgroups of a pass over 64 trials
constexpr uint32_t kColBins = 256;
constexpr uint64_t kColFloors = 32u << 20;      // values (of P) from which floors pay
constexpr uint32_t kColSmall = 36u << 10;   // nodes whose column one workgroup holds in LDS
constexpr uint32_t kColPad = kWave + 1;   // LDS words from one bin to the next
constexpr size_t kColLds = size_t(kColBins) * (kColPad + 1) * 4;

struct ColState {
  uint32_t lo, w, need, done;   // done: the sum takes the values above lo and `need` copies of lo
};

struct ColArgs {
  const int32_t* P;
  const uint32_t* deg;
  uint32_t n, t, k, parts;
  ColState* st;      // [t + 1], the degrees last
  uint32_t* cnt;     // [t + 1][parts][kColBins]
  uint64_t* sum;     // [t + 1][parts]
  int64_t* topk_sum;
  int64_t* deg_topk;
};

// 8 bins per octave (as the greedy's gain_bin), and the values of a bin:
// [lo, lo + 2^w).
__device__ __forceinline__ uint32_t col_bin(uint32_t x) {
  const uint32_t bl = 32u - __clz(x);
  return (bl - 1) * 8 + (bl >= 4 ? (x >> (bl - 4)) & 7u : (x << (4 - bl)) & 7u);
}
__device__ __forceinline__ void col_range(uint32_t bin, uint32_t* lo, uint32_t* w) {
  const uint32_t bl = bin / 8 + 1, sub = bin % 8;
  *w = bl >= 4 ? bl - 4 : 0u;
  *lo = bl >= 4 ? (8u + sub) << (bl - 4) : (8u + sub) >> (4 - bl);
}

// Calls row(u, deg[u]) for the nodes of the wave's share with degree above
// `above` (kRows rows under way at once), deg(d) with every lane's degrees.
template <typename Deg, typename Row>
__device__ __forceinline__ void col_nodes(const ColArgs& a, uint32_t above, const Deg& deg, const Row& row) {
  const uint64_t stride = uint64_t(gridDim.x) * kColBlock;
  for (uint64_t u0 = uint64_t(blockIdx.x) * kColBlock + (threadIdx.x & ~63u); u0 < a.n; u0 += stride) {
    const uint64_t u = u0 + lane_id();
    const uint32_t d = u < a.n ? a.deg[u] : 0u;
    deg(d);
    constexpr int kRows = 8;
    for (uint64_t m = __ballot(d > above); m;) {
      uint32_t at[kRows];
      int cnt = 0;
#pragma unroll
      for (int i = 0; i < kRows; ++i) {
        at[i] = m ? static_cast<uint32_t>(__ffsll(static_cast<unsigned long long>(m)) - 1) : 0u;
        cnt += m ? 1 : 0;
        m &= m - 1;
      }
      int32_t p[kRows];
#pragma unroll
      for (int i = 0; i < kRows; ++i) p[i] = i < cnt ? row.load(u0 + at[i]) : 0;
#pragma unroll
      for (int i = 0; i < kRows; ++i)
        if (i < cnt) row.use(2 * p[i] - static_cast<int32_t>(lane_u32(d, static_cast<int>(at[i]))));
    }
  }
}

// A lane's column of P and what becomes of its values.
template <typename F>
struct ColRow {
  const int32_t* P;
  uint32_t t, j;
  const F& f;
  __device__ __forceinline__ int32_t load(uint64_t u) const { return j < t ? P[u * t + j] : 0; }
  __device__ __forceinline__ void use(int32_t x) const {
    if (j < t && x > 0) f(static_cast<uint32_t>(x));
  }
};

// One counting pass for the trials 64 g .. 64 g + 63 of group g = blockIdx.y
// (and, in group 0, the degrees).
// pass 0: all values above the columns' floors; < 0: those of nodes of at least
// `some` entries, for the floors; > 0: those in the open ranges.
__global__ __launch_bounds__(kColBlock) void k_col_count(ColArgs a, int pass, uint32_t some) {
  extern __shared__ uint32_t col_lds[];
  uint32_t* hist = col_lds;                        // [bin][kColPad]
  uint32_t* dhist = col_lds + kColBins * kColPad;  // [bin]
  const uint32_t g = blockIdx.y, j = 64 * g + lane_id();
  const bool live = j < a.t, degs = g == 0;
  const ColState s = live ? a.st[j] : ColState{0, 0, 0, 1}, sd = degs ? a.st[a.t] : ColState{0, 0, 0, 1};
  if (__ballot(!s.done) == 0 && sd.done) return;   // uniform: every wave holds the same columns
  for (uint32_t i = threadIdx.x; i < kColBins * (kColPad + 1); i += kColBlock) col_lds[i] = 0;
  // a node below every open range is of no use
  const bool first = pass <= 0;
  uint32_t above = s.done ? 0xFFFFFFFFu : s.lo ? s.lo - 1 : 0u;
  if (pass < 0) above = some - 1;
  for (int o = 32; o; o >>= 1) above = min(above, static_cast<uint32_t>(__shfl_xor(static_cast<int>(above), o, kWave)));
  __syncthreads();
  const uint32_t lane = lane_id();
  const uint32_t shift = s.w > 8 ? s.w - 8 : 0u, dshift = sd.w > 8 ? sd.w - 8 : 0u;
  const auto count = [&](uint32_t x) {
    if (first)
      atomicAdd(&hist[col_bin(x) * kColPad + lane], 1u);
    else if (!s.done && x >= s.lo && (x - s.lo) >> s.w == 0)
      atomicAdd(&hist[((x - s.lo) >> shift) * kColPad + lane], 1u);
  };
  col_nodes(
      a, above,
      [&](uint32_t d) {
        if (!degs || d == 0) return;
        if (pass < 0 && d < some) return;
        if (first)
          atomicAdd(&dhist[col_bin(d)], 1u);
        else if (!sd.done && d >= sd.lo && (d - sd.lo) >> sd.w == 0)
          atomicAdd(&dhist[(d - sd.lo) >> dshift], 1u);
      },
      ColRow<decltype(count)>{a.P, a.t, j, count});
  __syncthreads();
  const uint32_t cols = a.t - 64 * g < 64 ? a.t - 64 * g : 64u;
  for (uint32_t i = threadIdx.x; i < cols * kColBins; i += kColBlock)
    a.cnt[(size_t(64 * g + i / kColBins) * a.parts + blockIdx.x) * kColBins + i % kColBins] =
        hist[(i % kColBins) * kColPad + i / kColBins];
  if (degs && threadIdx.x < kColBins)
    a.cnt[(size_t(a.t) * a.parts + blockIdx.x) * kColBins + threadIdx.x] = dhist[threadIdx.x];
}

// Narrows s by a pass's counts (one wave; cnt(bin) in any lane).  floor_only:
// the counts are of some of the column's values only, so the bin found bounds
// the k-th largest from below.
template <typename Cnt>
__device__ __forceinline__ void col_narrow(ColState& s, bool first, bool floor_only, const Cnt& cnt) {
  // lane l takes the bins 255 - 4 l, ..., 252 - 4 l: from the top
  constexpr uint32_t kOwn = kColBins / kWave;
  const uint32_t lane = lane_id();
  uint32_t h[kOwn], mine = 0;
#pragma unroll
  for (uint32_t i = 0; i < kOwn; ++i) {
    h[i] = cnt(kColBins - 1 - (lane * kOwn + i));
    mine += h[i];
  }
  uint32_t run = wave_incl_scan_u32(mine) - mine;
  const uint64_t hit = __ballot(run < s.need && s.need <= run + mine);
  if (!hit) {   // (the first pass) fewer than k positive values: all of them count
    if (!floor_only) s = ColState{0, 0, 0, 1};
    return;
  }
  uint32_t i = 0;
  while (i + 1 < kOwn && run + h[i] < s.need) run += h[i++];
  const int at = __ffsll(static_cast<unsigned long long>(hit)) - 1;
  const uint32_t b = lane_u32(kColBins - 1 - (lane * kOwn + i), at);
  run = lane_u32(run, at);
  if (floor_only) {
    uint32_t w;
    col_range(b, &s.lo, &w);
    return;
  }
  s.need -= run;
  if (first) {
    col_range(b, &s.lo, &s.w);
  } else {
    const uint32_t shift = s.w > 8 ? s.w - 8 : 0u;
    s.lo += b << shift;
    s.w = shift;
  }
  s.done = s.w == 0 ? 1u : 0u;
}

// Narrows column blockIdx.x's range by the pass's counts.
__global__ __launch_bounds__(kColBlock) void k_col_decide(ColArgs a, int pass) {
  __shared__ uint32_t part[kColBlock / kColBins][kColBins];
  const uint32_t c = blockIdx.x, bin = threadIdx.x % kColBins, q = threadIdx.x / kColBins;
  ColState s = a.st[c];
  if (s.done) return;
  uint32_t sum = 0;
  for (uint32_t p = q; p < a.parts; p += kColBlock / kColBins) sum += a.cnt[(size_t(c) * a.parts + p) * kColBins + bin];
  part[q][bin] = sum;
  __syncthreads();
  if (threadIdx.x >= kWave) return;
  col_narrow(s, pass == 0, pass < 0, [&](uint32_t b) {
    uint32_t x = 0;
    for (uint32_t i = 0; i < kColBlock / kColBins; ++i) x += part[i][b];
    return x;
  });
  if (threadIdx.x == 0) a.st[c] = s;
}

// The same for a column that fits in LDS: one workgroup per column reads it
// once.  (n = 2,000, t = 10: 57 us with R written by trial and selected by
// rows, ten launches, 4.5 so; n = 20,011, t = 32: 60, 27.)
__global__ __launch_bounds__(kColBlock) void k_col_small(ColArgs a) {
  extern __shared__ uint32_t col_lds[];   // the column's positive values, 0 for the others
  __shared__ uint32_t hist[kColBins];
  __shared__ uint64_t red[kColBlock / kWave];
  __shared__ ColState shared;
  const uint32_t c = blockIdx.x;
  ColState s{0, 0, a.k, 0};
  if (threadIdx.x < kColBins) hist[threadIdx.x] = 0;
  __syncthreads();
  for (uint32_t u = threadIdx.x; u < a.n; u += kColBlock) {
    const int32_t d = static_cast<int32_t>(a.deg[u]);
    const int32_t x = c < a.t ? 2 * a.P[uint64_t(u) * a.t + c] - d : d;
    col_lds[u] = x > 0 ? static_cast<uint32_t>(x) : 0u;
    if (x > 0) atomicAdd(&hist[col_bin(static_cast<uint32_t>(x))], 1u);
  }
  for (bool first = true;; first = false) {
    __syncthreads();
    if (threadIdx.x < kWave) {
      col_narrow(s, first, false, [&](uint32_t b) { return hist[b]; });
      if (threadIdx.x == 0) shared = s;
    }
    __syncthreads();
    s = shared;
    if (s.done) break;
    if (threadIdx.x < kColBins) hist[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t shift = s.w > 8 ? s.w - 8 : 0u;
    for (uint32_t u = threadIdx.x; u < a.n; u += kColBlock) {
      const uint32_t x = col_lds[u];
      if (x >= s.lo && (x - s.lo) >> s.w == 0) atomicAdd(&hist[(x - s.lo) >> shift], 1u);   // (s.lo >= 16)
    }
  }
  uint64_t sum = 0;
  for (uint32_t u = threadIdx.x; u < a.n; u += kColBlock) sum += col_lds[u] > s.lo ? col_lds[u] : 0u;
  sum = block_sum_u64<kColBlock>(sum, red);
  if (threadIdx.x) return;
  const int64_t r = static_cast<int64_t>(sum + uint64_t(s.need) * s.lo);
  if (c < a.t)
    a.topk_sum[c] = r;
  else
    *a.deg_topk = r;
}

// Sums of the values above lo.
__global__ __launch_bounds__(kColBlock) void k_col_sum(ColArgs a) {
  __shared__ unsigned long long sum[kWave], dsum;
  const uint32_t g = blockIdx.y, j = 64 * g + lane_id();
  const bool live = j < a.t, degs = g == 0;
  const uint32_t lo = live ? a.st[j].lo : 0xFFFFFFFFu, dlo = degs ? a.st[a.t].lo : 0xFFFFFFFFu;
  uint32_t above = lo;
  for (int o = 32; o; o >>= 1) above = min(above, static_cast<uint32_t>(__shfl_xor(static_cast<int>(above), o, kWave)));
  if (threadIdx.x < kWave) sum[threadIdx.x] = 0;
  if (threadIdx.x == 0) dsum = 0;
  __syncthreads();
  uint64_t acc = 0, dacc = 0;
  const auto add = [&](uint32_t x) { acc += x > lo ? x : 0u; };
  col_nodes(a, above, [&](uint32_t d) { dacc += d > dlo ? d : 0u; }, ColRow<decltype(add)>{a.P, a.t, j, add});
  if (acc) atomicAdd(&sum[lane_id()], static_cast<unsigned long long>(acc));
  if (dacc) atomicAdd(&dsum, static_cast<unsigned long long>(dacc));
  __syncthreads();
  if (threadIdx.x < kWave && live) a.sum[size_t(j) * a.parts + blockIdx.x] = sum[threadIdx.x];
  if (threadIdx.x == 0 && degs) a.sum[size_t(a.t) * a.parts + blockIdx.x] = dsum;
}

__global__ __launch_bounds__(kWave) void k_col_out(ColArgs a) {
  const uint32_t c = blockIdx.x;
  uint64_t sum = 0;
  for (uint32_t p = threadIdx.x; p < a.parts; p += kWave) sum += a.sum[size_t(c) * a.parts + p];
  sum = wave_sum_u64(sum);
  if (threadIdx.x) return;
  const ColState s = a.st[c];
  const int64_t r = static_cast<int64_t>(sum + uint64_t(s.need) * s.lo);
  if (c < a.t)
    a.topk_sum[c] = r;
  else
    *a.deg_topk = r;
}

__global__ void k_col_init(ColArgs a) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c <= a.t) a.st[c] = ColState{0, 0, a.k, 0};
}

static uint32_t col_parts(uint32_t n, uint32_t t) {
  const uint32_t groups = (t + 63) / 64, most = kColParts / groups ? kColParts / groups : 1u;
  const uint32_t want = (n + kColBlock - 1) / kColBlock;
  return want < most ? want : most;
}

static size_t col_ws_bytes(uint32_t n, uint32_t t) {
  return size_t(t + 1) * (sizeof(ColState) + size_t(col_parts(n, t)) * (kColBins * 4 + 8));
}

// The most that any number of trials up to t takes: a group of 64 more
// leaves each group fewer workgroups (n = 10^6: 64 trials 17.2 MB, 65 trials
// 8.8 MB, 100 trials 13.3 MB).
static size_t col_ws_most(uint32_t n, uint32_t t) {
  size_t most = col_ws_bytes(n, t);
  for (uint32_t full = 64; full < t; full += 64) most = std::max(most, col_ws_bytes(n, full));
  return most;
}

// max_value: a bound on the degrees.
static void columns_topk(const int32_t* P, const uint32_t* deg, uint32_t n, uint32_t t, uint32_t k, uint64_t max_value,
                         void* ws, int64_t* topk_sum, int64_t* deg_topk, hipStream_t s) {
  ColArgs a{};
  a.P = P;
  a.deg = deg;
  a.n = n;
  a.t = t;
  a.k = k;
  a.parts = col_parts(n, t);
  a.sum = static_cast<uint64_t*>(ws);
  a.st = reinterpret_cast<ColState*>(a.sum + size_t(t + 1) * a.parts);
  a.cnt = reinterpret_cast<uint32_t*>(a.st + (t + 1));
  a.topk_sum = topk_sum;
  a.deg_topk = deg_topk;
  const dim3 grid(a.parts, (t + 63) / 64), block(kColBlock);
  if (n <= kColSmall) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_col_small), hipFuncAttributeMaxDynamicSharedMemorySize,
                              static_cast<int>(kColSmall * 4));
    hipLaunchKernelGGL(k_col_small, dim3(t + 1), block, size_t(n) * 4, s, a);
    return;
  }
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_col_count), hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(kColLds));
  hipLaunchKernelGGL(k_col_init, dim3((t + 256) / 256), dim3(256), 0, s, a);
  // Floors for the columns' k-th values from the nodes of several times the
  // mean degree, which on skewed samples rule most rows out of the first pass.
  // They cost a pass over the degrees and two launches, 25 us, and spare up to
  // the reading of P (n = 10^6, t = 64: 735 us for the whole call without, 677
  // with; n = 10^5: 5 us more).
  if (uint64_t(n) * t >= kColFloors) {
    const uint64_t mean = max_value / n;
    const uint32_t some = mean < (1u << 26) ? static_cast<uint32_t>(4 * mean + 8) : 1u << 28;
    hipLaunchKernelGGL(k_col_count, grid, block, kColLds, s, a, -1, some);
    hipLaunchKernelGGL(k_col_decide, dim3(t + 1), block, 0, s, a, -1);
  }
  // the first pass leaves ranges of at most 2^(bits - 4) values, each further
  // one 2^8 times less
  int bits = 0;
  while (bits < 31 && max_value >> bits) ++bits;
  for (int left = bits > 4 ? bits - 4 : 0, pass = 0; pass == 0 || left > 0; ++pass) {
    hipLaunchKernelGGL(k_col_count, grid, block, kColLds, s, a, pass, 0u);
    hipLaunchKernelGGL(k_col_decide, dim3(t + 1), block, 0, s, a, pass);
    if (pass) left -= 8;
  }
  hipLaunchKernelGGL(k_col_sum, grid, block, 0, s, a);
  hipLaunchKernelGGL(k_col_out, dim3(t + 1), dim3(kWave), 0, s, a);
}

int mcera_reserve(centra_ctx* ctx, uint32_t n, uint64_t m, uint32_t t, hipStream_t s) {
  const uint32_t Wt = (t + 63) / 64;
  int rc;
  if ((rc = ensure(ctx, ctx->words, size_t(m) * Wt * 8, true, s))) return rc;
  if ((rc = ensure(ctx, ctx->P, size_t(n) * t * 4, true, s))) return rc;
  if ((rc = ensure(ctx, ctx->topk_tmp, col_ws_most(n, t), false, s))) return rc;
  return ensure(ctx, ctx->ext_bmax, 256, true, s);
}

int mcera_on_incidence(centra_ctx* ctx, uint32_t n, uint64_t m, uint64_t m0, const uint64_t* he_off, uint32_t t,
                       uint32_t k, int64_t* topk_sum, uint64_t* deg_topk, uint32_t* b_max, int32_t* R_out,
                       hipStream_t s) {
  // samples [m0, m) are counted: entries [he_off[m0], he_off[m]) of the
  // incidence, at most the newest segment's span when that is where m0 is
  const uint64_t span_cap = m0 == ctx->inc_m0 ? ctx->inc_span_cap : ctx->inc_limit;
  int rc;
  if ((rc = ensure(ctx, ctx->P, size_t(n) * t * 4, m0 > 0, s))) return rc;
  if ((rc = ensure(ctx, ctx->topk_tmp, col_ws_bytes(n, t), false, s))) return rc;
  int32_t* P = static_cast<int32_t*>(ctx->P.ptr);
  const uint32_t* deg = static_cast<const uint32_t*>(ctx->deg.ptr);
  if (m0 == 0) fill_u32(reinterpret_cast<uint32_t*>(P), 0, size_t(n) * t, s);
  rade_count_launch(static_cast<const uint32_t*>(ctx->inc.ptr), static_cast<const uint32_t*>(ctx->inc_node.ptr), he_off,
                    m0, m, span_cap, ctx->inc_limit, static_cast<const uint64_t*>(ctx->words.ptr), t,
                    m0 == 0 && ctx->inc_nseg == 1, P, s);
  if (R_out)
    hipLaunchKernelGGL(k_rade_rows, dim3(grid_for(uint64_t(n) * t, 256)), dim3(256), 0, s, P, deg, n, t, R_out);
  columns_topk(P, deg, n, t, k, ctx->inc_limit, ctx->topk_tmp.ptr, topk_sum, reinterpret_cast<int64_t*>(deg_topk), s);
  if (m0 == 0) fill_u32(b_max, 0, 1, s);
  if (m > m0)
    hipLaunchKernelGGL(k_bmax, dim3(grid_for(m - m0, kBmaxBlock, 512)), dim3(kBmaxBlock), 0, s, he_off + m0, m - m0,
                       b_max);
  CENTRA_HIP(ctx, hipGetLastError());
  return CENTRA_OK;
}

}  // namespace centra
