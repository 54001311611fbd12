// stream_common.hpp -- building blocks of the index-stream kernels (the
// delta-varint and 2-D COO encoders and decoders): reduce-then-scan over tiles
// of a stream whose length is read from the device.
//
//   1. reduce  one block per tile folds its part of the stream into an
//              aggregate, kept in the workspace's table words;
//   2. write   one block per tile starts from the fold of the aggregates
//              before its own, reads its part again and writes its output.
// The encoders' blocks fold plain sums themselves (a few words per thread cost
// less than a launch); the decoders have a small launch in between.  Every word is
// written before it is read, so what a batch's tensor table left there does not
// matter, and the words a call used are left zero.  No block waits on another.
#pragma once

#include "device_common.hpp"

namespace pulse {
namespace stream {

constexpr int kDT = 256;                     // threads per block of the tile kernels
constexpr int kDWaves = kDT / 64;
constexpr uint32_t kDUnit = kDT * 16;        // bytes (varint) or pairs (COO) per unit
// Tiles per launch, up to three table words each.  More cost the fold of the
// tile words in every block, fewer leave the last wave of tiles longer: 2,047 /
// 4,095 / 8,191 took 370 / 355 / 365 us on the 7B set's varint stream (encode
// and decode) and 89 / 90 / 92 us on the 0.5B set's COO stream.
constexpr uint32_t kMaxStreamTiles = 4095;
constexpr int kST = 1024;                    // threads of the single-block scan
static_assert(3 * (uint64_t)(kMaxStreamTiles + 1) <= kTableWords, "tile aggregates exceed the table");
// Tile aggregates a thread folds for its block's prefix.
constexpr uint32_t kFoldPer = (kMaxStreamTiles + kDT) / kDT;

__device__ __forceinline__ uint64_t* stream_words(uint64_t* ws) { return ws + kTableOffsetWords; }

// LDS arrays that threads fill sixteen consecutive items each (thread t at
// 16 t + j) get one spare word per sixteen: item i lives at pad(i), so the 64
// lanes of a wave hit 64 different banks instead of four.
__device__ __forceinline__ uint32_t pad(uint32_t i) { return i + (i >> 4); }
constexpr uint32_t padded(uint32_t n) { return n + n / 16 + 1; }

// Tiles of a stream of n units' worth of items: each tile holds `per` units;
// at least one tile (an empty stream still has segments to finish).
struct Geo {
  uint64_t tile;    // items per tile
  uint32_t ntiles;
};

__device__ __forceinline__ Geo stream_geometry(uint64_t n) {
  const uint64_t units = n == 0 ? 1 : (n + kDUnit - 1) / kDUnit;
  const uint64_t per = (units + kMaxStreamTiles - 1) / kMaxStreamTiles;
  Geo g;
  g.tile = per * kDUnit;
  g.ntiles = (uint32_t)((units + per - 1) / per);
  return g;
}

// ---------------------------------------------------------------- block scans
//
// Exclusive scan over the threads of a block, in thread order, of an
// associative operation comb(earlier, later) with identity T::id(); `carry`
// comes before thread 0.  *total receives carry combined with every thread's
// value.  Every thread of the block calls it; s_w holds one value per wave.

template <int NT, typename T>
__device__ T block_scan_excl(T v, T carry, T* s_w, T* total) {
  const int lane = lane_id(), wid = (int)threadIdx.x >> 6;
  T inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const T o = shfl_up(inc, d);
    if (lane >= d) inc = comb(o, inc);
  }
  const T before = shfl_up(inc, 1);
  if (lane == 63) s_w[wid] = inc;
  __syncthreads();
  T pre = carry, all = carry;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const T x = s_w[w];
    if (w < wid) pre = comb(pre, x);
    all = comb(all, x);
  }
  __syncthreads();  // s_w may be reused
  *total = all;
  return lane == 0 ? pre : comb(pre, before);
}

// Block-wide exclusive sum of one count per thread (thread order).
__device__ inline uint32_t block_count_excl(uint32_t v, uint32_t* s_w, uint32_t* total) {
  const int lane = lane_id(), wid = (int)threadIdx.x >> 6;
  const uint32_t incl = wave_incl_scan(v);
  if (lane == 63) s_w[wid] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kDWaves; ++w) {
    const uint32_t x = s_w[w];
    if (w < wid) before += x;
    all += x;
  }
  __syncthreads();
  *total = all;
  return before + incl - v;
}

// First position in [0, n) with a(pos) >= key (a non-decreasing), whole wave.
template <typename At>
__device__ uint32_t lower_bound_wave(At a, uint32_t n, uint64_t key) {
  const int lane = lane_id();
  uint32_t lo = 0, hi = n;
  while (hi - lo > 64) {
    const uint32_t span = hi - lo;
    const uint32_t q = lo + (uint32_t)((uint64_t)span * (uint32_t)(lane + 1) / 65u);
    const uint64_t ge = __ballot(a(q) >= key);
    if (ge == 0) {
      lo = (uint32_t)__shfl((int)q, 63, 64) + 1;
    } else {
      const int f = __builtin_ctzll(ge);
      const uint32_t qf = (uint32_t)__shfl((int)q, f, 64);
      lo = f > 0 ? (uint32_t)__shfl((int)q, f - 1, 64) + 1 : lo;
      hi = qf;
    }
  }
  const uint32_t q = lo + (uint32_t)lane;
  const uint64_t ge = __ballot(q < hi && a(q) >= key);
  return ge == 0 ? hi : lo + (uint32_t)__builtin_ctzll(ge);
}

__device__ inline uint32_t lower_bound_wave(const uint64_t* a, uint32_t n, uint64_t key) {
  return lower_bound_wave([a](uint32_t i) { return a[i]; }, n, key);
}

// ---------------------------------------------------------------- segment starts
//
// A tile reads the segments that start in it once (one wave search), into LDS;
// its units then mark their starts and find an item's segment from LDS, with
// no dependent global load on a unit's path.

constexpr uint32_t kSegCache = kDT;  // starts kept per tile; more are read from memory

struct SegCache {
  uint64_t start[kSegCache];
  uint32_t lo;   // first segment starting at or after the tile's first item
  uint32_t n;    // segments starting in the tile
};

// Segments starting in [t0, t1) (starts non-decreasing; NULL: none).  Every
// thread calls it; it ends with a barrier.
__device__ inline void cache_tile_segments(const uint64_t* starts, uint32_t nseg, uint64_t t0,
                                           uint64_t t1, SegCache& C) {
  if (threadIdx.x < 64) {
    const uint32_t lane = (uint32_t)lane_id();
    uint32_t lo = 0, n = 0;
    if (starts && nseg > 0 && t1 > t0) {
      lo = lower_bound_wave(starts, nseg, t0);
      for (uint32_t m = 0;; m += 64) {
        const uint32_t s = lo + m + lane;
        const uint64_t v = s < nseg ? starts[s] : 0;
        const bool in = s < nseg && v < t1;
        if (in && m + lane < kSegCache) C.start[m + lane] = v;
        const uint64_t b = __ballot(in);
        n += (uint32_t)__builtin_popcountll(b);
        if (b != ~0ull) break;
      }
    }
    if (lane == 0) {
      C.lo = lo;
      C.n = n;
    }
  }
  __syncthreads();
}

// Start of segment s, s in [C.lo, C.lo + C.n).  (The read from memory, for
// starts past the cache, is a relaxed atomic load so that the compiler keeps
// it apart from the LDS read instead of merging both into one load through a
// generic pointer, which gfx950 code generation rejects here.)
__device__ __forceinline__ uint64_t start_of(const uint64_t* starts, const SegCache& C, uint32_t s) {
  const uint32_t i = s - C.lo;
  if (i < kSegCache) return C.start[i];
  return __hip_atomic_load(starts + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// First segment of the tile's with start >= key (C.lo + C.n if none).
__device__ inline uint32_t lower_bound_cached(const uint64_t* starts, const SegCache& C, uint64_t key) {
  uint32_t lo = 0, hi = C.n;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (start_of(starts, C, C.lo + mid) < key) lo = mid + 1;
    else hi = mid;
  }
  return C.lo + lo;
}

__device__ __forceinline__ bool bit_at(const uint32_t* s_bits, uint32_t i) {
  return (s_bits[i >> 5] >> (i & 31)) & 1u;
}

// The segment holding item k: the last segment starting at or before k, among
// [lo, hi) (those starting in the unit, all cached or in memory), else the one
// before lo (0 if none).
__device__ __forceinline__ uint32_t segment_of(const uint64_t* starts, const SegCache& C, uint32_t lo,
                                               uint32_t hi, uint64_t k) {
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (start_of(starts, C, mid) <= k) lo = mid + 1;
    else hi = mid;
  }
  return lo > 0 ? lo - 1 : 0;
}

// Sum of 64-bit values, for block_scan_excl.
struct Sum64 {
  uint64_t v;
  __device__ static Sum64 id() { return Sum64{0ull}; }
};
__device__ __forceinline__ Sum64 comb(Sum64 x, Sum64 y) { return Sum64{x.v + y.v}; }
__device__ __forceinline__ Sum64 shfl_up(Sum64 x, int d) { return Sum64{__shfl_up(x.v, d, 64)}; }

// Exclusive scan of n elements in place by one block of kST threads: each
// thread folds a run of consecutive elements, the runs are scanned, and each
// thread writes its run's prefixes.
template <typename T, typename Load, typename Store>
__device__ void single_block_scan(uint32_t n, Load ld, Store st, T* s_w) {
  const uint32_t per = (n + kST - 1) / kST;
  const uint32_t a = (uint32_t)threadIdx.x * per;
  const uint32_t b = a + per < n ? a + per : n;
  T run = T::id();
  for (uint32_t i = a; i < b; ++i) run = comb(run, ld(i));
  T all;
  T pre = block_scan_excl<kST>(run, T::id(), s_w, &all);
  for (uint32_t i = a; i < b; ++i) {
    const T x = ld(i);
    st(i, pre);
    pre = comb(pre, x);
  }
}

// Sum of w[0 .. n), n <= kMaxStreamTiles; every thread of the block gets it.
// s_w holds one value per wave; contains one barrier, and s_w may be reused
// after the next.
__device__ __forceinline__ uint64_t fold_before(const uint64_t* w, uint32_t n, uint64_t* s_w) {
  uint64_t v = 0;
#pragma unroll
  for (uint32_t q = 0; q < kFoldPer; ++q) {
    const uint32_t i = q * kDT + threadIdx.x;
    if (i < n) v += w[i];
  }
  v = wave_sum_u64(v);
  if (lane_id() == 0) s_w[threadIdx.x >> 6] = v;
  __syncthreads();
  uint64_t all = 0;
#pragma unroll
  for (int q = 0; q < kDWaves; ++q) all += s_w[q];
  return all;
}

// Called by every block of a write pass at its end, by all threads: counts the
// block out, and the last one out -- every block has read its aggregates --
// clears words [0, n0).  Relaxed: a block's reads have
// returned (the wait) before it counts itself out, and nothing else is ordered.
__device__ __forceinline__ void stream_finish(uint64_t* ws, uint32_t ntiles, uint32_t n0) {
  if (threadIdx.x >= 64) return;
  uint32_t last = 0;
  if (threadIdx.x == 0) {
    __builtin_amdgcn_s_waitcnt(0);  // every counter at zero
    last = __hip_atomic_fetch_add(ws + kWordStream, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           ntiles - 1;
    if (last) __hip_atomic_store(ws + kWordStream, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!__builtin_amdgcn_readfirstlane((int)last)) return;
  uint64_t* w = stream_words(ws);
  for (uint32_t i = threadIdx.x; i < n0; i += 64) w[i] = 0;
}

// Prefetches.  A load that one of two paths issues, or that a branch skips, has
// its registers merged where the paths join, and the compiler waits for it
// there -- right after issuing it.  Every prefetch below is therefore one
// unconditional load per register, from the stream or (for lanes without a
// whole piece in range) from a zero block; the one ragged piece at a list's
// end is read again, item by item, when its unit is computed.
__device__ __align__(16) const uint32_t kStreamZero[4] = {0u, 0u, 0u, 0u};

// A unit's entries as its threads hold them: four quads of four consecutive
// entries, quad q of thread t the entries 4 (q kDT + t) .. + 3 of the unit, so
// that each load instruction reads whole lines.  Entries at or past u1 read as
// 0.  The 16-byte loads need the list's own 4-byte alignment only.
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

struct Quads {
  uint32_t v[16];   // quad q's entries at 4 q ..
  uint32_t edge[4]; // lane 0: the entry before quad q (0 before the list)
};

__device__ __forceinline__ Quads load_quads(const uint32_t* idx, uint64_t u0, uint64_t u1) {
  Quads x;
  const uint32_t* const zero = kStreamZero;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint64_t k = u0 + 4ull * ((uint32_t)q * kDT + threadIdx.x);
    const u32x4_a4 w = *reinterpret_cast<const u32x4_a4*>(k + 4 <= u1 ? idx + k : zero);
    x.v[4 * q] = w.x;
    x.v[4 * q + 1] = w.y;
    x.v[4 * q + 2] = w.z;
    x.v[4 * q + 3] = w.w;
    x.edge[q] = *(lane_id() == 0 && k > 0 && k < u1 ? idx + k - 1 : zero);
  }
  return x;
}

// The ragged quad of a unit [u0, u1) that ends the list.
__device__ __forceinline__ void finish_quads(Quads& x, const uint32_t* idx, uint64_t u0, uint64_t u1) {
  if (u1 - u0 == kDUnit) return;  // block-uniform
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint64_t k = u0 + 4ull * ((uint32_t)q * kDT + threadIdx.x);
    if (k < u1 && k + 4 > u1) {
#pragma unroll
      for (int j = 0; j < 3; ++j) x.v[4 * q + j] = k + j < u1 ? idx[k + j] : 0u;
    }
  }
}

// The entry before quad q: the previous lane's last, or the edge (wave_shr:1
// keeps lane 0's own value).
__device__ __forceinline__ uint32_t before_quad(const Quads& x, int q) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)x.edge[q], (int)x.v[4 * q + 3], 0x138, 0xF, 0xF, false);
}

// Entries of quad q below u1 (0 to 4).
__device__ __forceinline__ uint32_t quad_len(uint64_t u0, uint64_t u1, int q) {
  const uint64_t k = u0 + 4ull * ((uint32_t)q * kDT + threadIdx.x);
  return k < u1 ? (uint32_t)(u1 - k < 4 ? u1 - k : 4) : 0u;
}

// Clears the bitmap and marks the items of [u0, u1) at which a segment starts,
// from the tile's cached starts; nothing for a tile without any.  Every thread
// calls it.  With starts in the tile it contains two barriers, the first after
// the bitmap's clearing.  (Item 0 of the list needs no mark of its own: the
// item before it reads as 0.)
__device__ __forceinline__ void mark_unit(const uint64_t* starts, const SegCache& C, uint64_t u0, uint64_t u1,
                                          uint32_t* bits) {
  if (C.n == 0) return;  // block-uniform
  for (uint32_t i = threadIdx.x; i < kDUnit / 32; i += kDT) bits[i] = 0;
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < C.n; i += kDT) {
    const uint64_t v = start_of(starts, C, C.lo + i);
    if (v >= u0 && v < u1) {
      const uint32_t b = (uint32_t)(v - u0);
      atomicOr(&bits[b >> 5], 1u << (b & 31));
    }
  }
  __syncthreads();
}

// Marks of this thread's quads (bit 4 q + j), and of its sixteen consecutive items.
__device__ __forceinline__ uint32_t quad_marks(const SegCache& C, const uint32_t* bits) {
  if (C.n == 0) return 0u;
  uint32_t m = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t i = 4u * ((uint32_t)q * kDT + threadIdx.x);
    m |= ((bits[i >> 5] >> (i & 31)) & 0xFu) << (4 * q);
  }
  return m;
}

__device__ __forceinline__ uint32_t run_marks(const SegCache& C, const uint32_t* bits) {
  if (C.n == 0) return 0u;
  return (bits[threadIdx.x >> 1] >> (16 * (threadIdx.x & 1))) & 0xFFFFu;
}

// Exclusive positions of a unit's quads in list order (quad 0 of every thread,
// then quad 1, ...) from their sizes (at most 2^16 / kDT each); *total receives
// the unit's.  One barrier; s_w is rewritten by the next call but one.
__device__ __forceinline__ void scan_quads(const uint32_t (&size)[4], uint2 (*s_w)[kDWaves], int parity,
                                           uint32_t (&at)[4], uint32_t* total) {
  const uint32_t a = size[0] | (size[1] << 16), b = size[2] | (size[3] << 16);
  const uint32_t ia = wave_incl_scan(a), ib = wave_incl_scan(b);
  const int wid = (int)threadIdx.x >> 6;
  if (lane_id() == 63) s_w[parity][wid] = make_uint2(ia, ib);
  __syncthreads();
  uint32_t ba = 0, bb = 0, ta = 0, tb = 0;
#pragma unroll
  for (int w = 0; w < kDWaves; ++w) {
    const uint2 x = s_w[parity][w];
    ba += w < wid ? x.x : 0u;
    bb += w < wid ? x.y : 0u;
    ta += x.x;
    tb += x.y;
  }
  const uint32_t ea = ba + ia - a, eb = bb + ib - b;
  const uint32_t t0 = ta & 0xFFFFu, t1 = t0 + (ta >> 16), t2 = t1 + (tb & 0xFFFFu);
  at[0] = ea & 0xFFFFu;
  at[1] = t0 + (ea >> 16);
  at[2] = t1 + (eb & 0xFFFFu);
  at[3] = t2 + (eb >> 16);
  *total = t2 + (tb >> 16);
}

// Grid of a tile kernel over a stream of at most `capacity` items.
inline uint32_t tile_grid(uint64_t capacity) {
  const uint64_t units = capacity == 0 ? 1 : (capacity + kDUnit - 1) / kDUnit;
  return (uint32_t)(units < kMaxStreamTiles ? units : kMaxStreamTiles);
}

}  // namespace stream
}  // namespace pulse
