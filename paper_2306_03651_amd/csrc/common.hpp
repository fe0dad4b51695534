// Device-side building blocks shared by the CentRA kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace centra {

constexpr uint32_t kUnseen = 0xFFFFFFFFu;
constexpr int kWave = 64;

// Error bits raised by kernels into the context's device flag word.
constexpr uint32_t kErrNodeRange = 1u;      // a hyperedge names a node >= n
constexpr uint32_t kErrBacktrack = 2u;      // no predecessor found (impossible on valid input)
constexpr uint32_t kErrGraph = 4u;          // malformed CSR
constexpr uint32_t kErrCapacity = 8u;       // a hyperedge store exceeds its stated capacity
constexpr uint32_t kErrOffsets = 16u;       // hyperedge offsets decrease

// ---------------------------------------------------------------------------
// Coherent accesses.  The per-BFS arrays are updated with device-scope
// atomics (performed in L2) by several waves at once; plain loads could be
// served from a stale line of the CU's vector L1, so every access to them
// goes through relaxed agent-scope atomic loads and stores.
__device__ __forceinline__ uint32_t ld_u32(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_u64(const uint64_t* p) {
  return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_u32(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_u64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The same at workgroup scope, for arrays that one workgroup alone touches
// during a launch (the per-BFS slot state).
__device__ __forceinline__ uint32_t wg_ld_u32(const uint32_t* p) {
  return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint64_t wg_ld_u64(const uint64_t* p) {
  return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void wg_st_u32(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void wg_st_u64(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// ---------------------------------------------------------------------------
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each two
// 64x64->128 products with the published multipliers; the key advances by
// the published Weyl constants after every round.
struct Block4 {
  uint64_t w0, w1, w2, w3;
};

//
// kRounds: rounds per pass of the loop.  The workgroup samplers draw a few
// words per sample from uniform state (scalar code), at several places of a
// large kernel: with all ten rounds laid out at each, k_sample_paths was 83
// KB of code, more than the instruction cache, and a pair draw cost 12 to 33
// us in instruction fetches.  They roll the rounds up (1); kernels that draw
// per thread keep them straight (10).
template <int kRounds = 10>
__device__ __forceinline__ Block4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                               uint64_t k0, uint64_t k1) {
  const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll kRounds
  for (int r = 0; r < 10; ++r) {
    const uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
    const uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
    const uint64_t n0 = hi1 ^ c1 ^ k0;
    const uint64_t n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
    k0 += W0;
    k1 += W1;
  }
  return Block4{c0, c1, c2, c3};
}

// Word stream with key (seed, 0) and counter (block, c1, c2, c3): blocks
// 0, 1, 2, ... consumed four words at a time.  Kept in registers; the
// selection avoids dynamic indexing (which would spill to scratch).
template <int kRounds>
struct WordStreamOf {
  uint64_t seed, c1, c2, c3;
  uint64_t next_block;
  uint32_t pos;
  Block4 buf;

  __device__ __forceinline__ WordStreamOf(uint64_t seed_, uint64_t c1_, uint64_t c2_, uint64_t c3_)
      : seed(seed_), c1(c1_), c2(c2_), c3(c3_), next_block(0), pos(4), buf{0, 0, 0, 0} {}

  __device__ __forceinline__ uint64_t next() {
    if (pos == 4) {
      buf = philox4x64_10<kRounds>(next_block, c1, c2, c3, seed, 0);
      ++next_block;
      pos = 0;
    }
    const uint32_t p = pos++;
    return p == 0 ? buf.w0 : (p == 1 ? buf.w1 : (p == 2 ? buf.w2 : buf.w3));
  }
};

using WordStream = WordStreamOf<10>;
using RolledWordStream = WordStreamOf<1>;

// (2^64 - W) mod W by shift and subtract: needed only when a draw's low
// half falls below W (once in 2^64 / W draws), so it is kept small, not fast.
__device__ __forceinline__ uint64_t reject_below(uint64_t W) {
  const uint64_t x = 0ull - W;
  uint64_t r = 0;
#pragma unroll 1
  for (int i = 63; i >= 0; --i) {
    const bool carry = (r >> 63) != 0;
    r = (r << 1) | ((x >> i) & 1ull);
    if (carry || r >= W) r -= W;
  }
  return r;
}

// Lemire's bounded draw in [0, W) (TOMACS 2019): high half of x*W, with the
// low half rejected below (2^64 - W) mod W.  W >= 1.
template <typename Stream>
__device__ __forceinline__ uint64_t bounded(Stream& st, uint64_t W) {
  uint64_t x = st.next();
  uint64_t lo = x * W;
  if (lo < W) {
    const uint64_t thr = reject_below(W);
    while (lo < thr) {
      x = st.next();
      lo = x * W;
    }
  }
  return __umul64hi(x, W);
}

// ---------------------------------------------------------------------------
// Wave (64-lane) helpers.
__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Wave scans and reductions by DPP: lane i takes in lane i - 1, 2, 4, 8 of
// its row of 16 (row_shr), then rows 1 and 3 the total of the row before
// (row_bcast 15), then the upper half that of the lower (row_bcast 31).  A
// lane without a source takes 0, the identity of every operation below.
// One VALU instruction per step and word, where a shuffle is an LDS
// permute: the samplers' many short reductions wait for nothing but these.
// Call with every lane of the wave active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp0_u32(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xf, ROWS == 0xf));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp0_u64(uint64_t v) {
  return (uint64_t(dpp0_u32<CTRL, ROWS>(static_cast<uint32_t>(v >> 32))) << 32) |
         dpp0_u32<CTRL, ROWS>(static_cast<uint32_t>(v));
}
// Inclusive prefix of an associative operation with identity 0.
template <typename Op>
__device__ __forceinline__ uint64_t wave_prefix_u64(uint64_t v, const Op& op) {
  v = op(v, dpp0_u64<0x111, 0xf>(v));
  v = op(v, dpp0_u64<0x112, 0xf>(v));
  v = op(v, dpp0_u64<0x114, 0xf>(v));
  v = op(v, dpp0_u64<0x118, 0xf>(v));
  v = op(v, dpp0_u64<0x142, 0xa>(v));
  v = op(v, dpp0_u64<0x143, 0xc>(v));
  return v;
}
template <typename Op>
__device__ __forceinline__ uint32_t wave_prefix_u32(uint32_t v, const Op& op) {
  v = op(v, dpp0_u32<0x111, 0xf>(v));
  v = op(v, dpp0_u32<0x112, 0xf>(v));
  v = op(v, dpp0_u32<0x114, 0xf>(v));
  v = op(v, dpp0_u32<0x118, 0xf>(v));
  v = op(v, dpp0_u32<0x142, 0xa>(v));
  v = op(v, dpp0_u32<0x143, 0xc>(v));
  return v;
}
// Value of lane l (uniform), in scalar registers.
__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int l) {
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l));
}
__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int l) {
  return (uint64_t(lane_u32(static_cast<uint32_t>(v >> 32), l)) << 32) | lane_u32(static_cast<uint32_t>(v), l);
}

// Inclusive prefix sums over the 64 lanes.
__device__ __forceinline__ uint64_t wave_incl_scan_u64(uint64_t v) {
  return wave_prefix_u64(v, [](uint64_t a, uint64_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
  return wave_prefix_u32(v, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) { return lane_u64(wave_incl_scan_u64(v), kWave - 1); }
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) { return lane_u32(wave_incl_scan_u32(v), kWave - 1); }
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
  return lane_u64(wave_prefix_u64(v, [](uint64_t a, uint64_t b) { return a > b ? a : b; }), kWave - 1);
}
// Workgroup-uniform values read from LDS or reduced across the block: the
// readfirstlane tells the compiler so, which keeps them (and what is derived
// from them) in scalar registers.  Only for values every lane holds equal.
__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(x)));
}
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
  return (uint64_t(uniform_u32(static_cast<uint32_t>(x >> 32))) << 32) | uniform_u32(static_cast<uint32_t>(x));
}

// Block-wide exclusive scan of one u32 per thread; *total gets the sum.
// `scratch` holds BLOCK/64 words of LDS.  Contains barriers.
template <int BLOCK>
__device__ __forceinline__ uint32_t block_excl_scan_u32(uint32_t v, uint32_t* total, uint32_t* scratch) {
  constexpr int NW = BLOCK / kWave;
  const int lane = lane_id(), wid = threadIdx.x / kWave;
  const uint32_t incl = wave_incl_scan_u32(v);
  if (lane == kWave - 1) scratch[wid] = incl;
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const uint32_t x = scratch[i];
    before += i < wid ? x : 0u;
    tot += x;
  }
  __syncthreads();
  *total = uniform_u32(tot);
  return before + incl - v;
}

template <int BLOCK>
__device__ __forceinline__ uint64_t block_max_u64(uint64_t v, uint64_t* scratch) {
  constexpr int NW = BLOCK / kWave;
  const int lane = lane_id(), wid = threadIdx.x / kWave;
  v = wave_max_u64(v);
  if (lane == 0) scratch[wid] = v;
  __syncthreads();
  uint64_t r = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) r = scratch[i] > r ? scratch[i] : r;
  __syncthreads();
  return uniform_u64(r);
}

template <int BLOCK>
__device__ __forceinline__ uint64_t block_sum_u64(uint64_t v, uint64_t* scratch) {
  constexpr int NW = BLOCK / kWave;
  const int lane = lane_id(), wid = threadIdx.x / kWave;
  v = wave_sum_u64(v);
  if (lane == 0) scratch[wid] = v;
  __syncthreads();
  uint64_t r = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) r += scratch[i];
  __syncthreads();
  return uniform_u64(r);
}

// Saturating u64 addition (for sums of which only "below 2^C" is asked).
__device__ __forceinline__ uint64_t sat_add(uint64_t a, uint64_t b) {
  const uint64_t c = a + b;
  return c < a ? ~0ull : c;
}

// Workgroup collectives with one barrier each.  The waves' partial results
// go to one of two halves of `buf` in turn: a wave that writes a half again
// has passed the barrier of the collective between, which every wave
// reaches only after its reads of that half, so no trailing barrier is
// needed.  Every thread of the workgroup calls them in the same order, and
// each orders the workgroup's memory accesses before it and after it as a
// barrier does.  A workgroup of one wave needs no LDS and no barrier: there
// __syncthreads only keeps the order.
template <int BLOCK>
struct Coll {
  static constexpr int NW = BLOCK / kWave;
  static constexpr int kHalf = 2 * NW;   // u64 words a collective may use
  uint64_t* buf;                         // LDS, 2 * kHalf words
  uint32_t at;                           // the half in turn (0 or kHalf)

  __device__ __forceinline__ uint64_t* turn() {
    at ^= kHalf;
    return buf + at;
  }
  template <typename Op>
  __device__ __forceinline__ uint64_t reduce(uint64_t v, const Op& op) {
    v = lane_u64(wave_prefix_u64(v, op), kWave - 1);
    if constexpr (NW > 1) {
      uint64_t* p = turn();
      if (lane_id() == 0) p[threadIdx.x / kWave] = v;
      __syncthreads();
      v = p[0];
#pragma unroll
      for (int i = 1; i < NW; ++i) v = op(v, p[i]);
      v = uniform_u64(v);
    } else {
      __syncthreads();
    }
    return v;
  }
  __device__ __forceinline__ uint64_t sum(uint64_t v) {
    return reduce(v, [](uint64_t a, uint64_t b) { return a + b; });
  }
  __device__ __forceinline__ uint64_t max(uint64_t v) {
    return reduce(v, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
  }
  __device__ __forceinline__ uint64_t sat_sum(uint64_t v) { return reduce(v, sat_add); }
  // the maximum of *mx and the saturating sum of *sum, with one barrier
  __device__ __forceinline__ void max_and_sat_sum(uint64_t* mx, uint64_t* sum) {
    const auto mop = [](uint64_t a, uint64_t b) { return a > b ? a : b; };
    uint64_t m = lane_u64(wave_prefix_u64(*mx, mop), kWave - 1);
    uint64_t s = lane_u64(wave_prefix_u64(*sum, sat_add), kWave - 1);
    if constexpr (NW > 1) {
      uint64_t* p = turn();
      const int wid = threadIdx.x / kWave;
      if (lane_id() == 0) {
        p[2 * wid] = m;
        p[2 * wid + 1] = s;
      }
      __syncthreads();
      m = p[0];
      s = p[1];
#pragma unroll
      for (int i = 1; i < NW; ++i) {
        m = mop(m, p[2 * i]);
        s = sat_add(s, p[2 * i + 1]);
      }
      m = uniform_u64(m);
      s = uniform_u64(s);
    } else {
      __syncthreads();
    }
    *mx = m;
    *sum = s;
  }
  __device__ __forceinline__ bool any(bool x) {
    bool r = __ballot(x) != 0;
    if constexpr (NW > 1) {
      uint64_t* p = turn();
      if (lane_id() == 0) p[threadIdx.x / kWave] = r ? 1u : 0u;
      __syncthreads();
      uint64_t any_set = p[0];
#pragma unroll
      for (int i = 1; i < NW; ++i) any_set |= p[i];
      r = uniform_u64(any_set) != 0;
    } else {
      __syncthreads();
    }
    return r;
  }
  // exclusive scans in thread order of a u32 per thread and of its being
  // nonzero; *total receives the sum
  __device__ __forceinline__ void scan_and_rank(uint32_t v, uint32_t* off, uint32_t* rank, uint32_t* total) {
    const uint32_t incl = wave_incl_scan_u32(v);
    const uint64_t m = __ballot(v != 0);
    uint32_t o = incl - v;
    uint32_t r = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                           __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0));
    uint32_t tot = lane_u32(incl, kWave - 1);
    if constexpr (NW > 1) {
      uint64_t* p = turn();
      const int wid = threadIdx.x / kWave;
      if (lane_id() == 0) p[wid] = uint64_t(__popcll(m)) << 32 | tot;
      __syncthreads();
      tot = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const uint64_t x = p[i];
        if (i < wid) {
          o += static_cast<uint32_t>(x);
          r += static_cast<uint32_t>(x >> 32);
        }
        tot += static_cast<uint32_t>(x);
      }
      tot = uniform_u32(tot);
    } else {
      __syncthreads();
    }
    *off = o;
    *rank = r;
    *total = tot;
  }
  // exclusive scan in thread order; *total receives the sum
  __device__ __forceinline__ uint64_t scan(uint64_t v, uint64_t* total) {
    const uint64_t incl = wave_incl_scan_u64(v);
    uint64_t before = 0, tot;
    if constexpr (NW > 1) {
      uint64_t* p = turn();
      const int wid = threadIdx.x / kWave;
      if (lane_id() == kWave - 1) p[wid] = incl;
      __syncthreads();
      tot = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const uint64_t x = p[i];
        before += i < wid ? x : 0ull;
        tot += x;
      }
      tot = uniform_u64(tot);
    } else {
      tot = lane_u64(incl, kWave - 1);
      __syncthreads();
    }
    *total = tot;
    return before + incl - v;
  }
};

__device__ __forceinline__ uint32_t bitlen64(uint64_t x) { return x ? 64u - __clzll(x) : 0u; }
__device__ __forceinline__ uint32_t bitlen32(uint32_t x) { return x ? 32u - __clz(x) : 0u; }

}  // namespace centra
