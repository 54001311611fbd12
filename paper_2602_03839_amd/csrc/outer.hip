// outer.hip -- PULSELoCo outer step on gfx950 (Sec. 4.3, Alg. 2: SparseSync
// and the outer Nesterov update).  SparseSync's result g is the union of the
// workers' selected entries, each the average over all R workers of the
// values sent (a worker that sent nothing counts as zero); then
//   m     <- mu * m + g
//   theta <- theta - alpha * (mu * m + g)
// with one FP32 rounding per operation.
//
// g is never materialised in HBM.  Each worker's list is sorted by index (the
// sparsifier writes it in index order), so a tile's entries are one run of it:
// a block finds the runs by search, adds them into an LDS copy of the tile's g
// -- worker by worker, with a barrier between workers, so every sum is formed
// in worker order -- and streams theta and m once, reading g from LDS.  HBM
// traffic: 8 bytes read and 8 written per element, 8 per list entry.
#include "device_common.hpp"
#include "launch.hpp"

namespace pulse {

namespace {

// What bounds it: HBM, as four streams (theta and m read and written), which
// blocks that each do one round of loads and stores carry fastest: 494M
// elements without lists take 1.30 ms (6.1 TB/s), against 1.59 ms for blocks
// that walk 262,144 elements each.  The lists add the searches' probes and
// latency.  Measured on the 218-tensor 0.5B set (ms, 2% density; 1, 4 and 8
// workers): 262,144-element units 1.66, 1.98-2.04, 2.64; this form 1.41, 1.42,
// 1.64.  Small sets gain more, since a unit was one block's work: 3M elements
// in 40 tensors with 8 workers 240 -> 32 us.
constexpr int kOuterTB = 512;                   // threads per block
constexpr int kOuterWaves = kOuterTB / 64;
constexpr int kOuterVec = 3;                    // float4 per thread
constexpr uint32_t kOuterTile = kOuterTB * kOuterVec * 4;  // elements of a block
// List entries of a tile a wave holds, per lane: kFirst loaded at once (128
// entries of 6,144 elements: 2% density), the rest only if the tile has more.
// Tiles of 4,096 or 8,192 elements were within 3% at 2% density and one to
// four workers; one wave per list needs eight waves for eight workers (four
// waves of 256-thread blocks: 1.94 ms with 8 workers).
constexpr int kFirst = 2;
constexpr int kHeld = 4;
static_assert(kOuterWaves >= kMaxLists, "one wave per list");
// Launches of up to this many tiles, a block per CU, take the SMALL form: less
// stands in front of a block's first list entries (the list's descriptor comes by
// scalar loads, and a tensor's first tile, which starts with the tensor's first
// entry, searches nothing).  Sets of many small tensors are bound by that latency:
// 500K elements in 300 tensors, one worker (five launches of ~75 tiles) 42.2 us,
// SMALL 38.0; 3M in 1,500 217, 189.  Past it the streams' order counts more: 5M in
// 40 tensors (830 tiles), one worker 16.0, SMALL 16.8; 100M in one, 282, 288; 400M,
// four workers 1,127, 1,179.
constexpr uint32_t kSmallTiles = 256;

// First position in [lo, hi) with idx >= target, or hi.  Whole wave.  `x`: the
// target's place in the tensor, in [0, 1].  Each round reads 16 probes (a probe
// costs a cache line: 64 of them per round moved more bytes than the tile
// itself), the first one around where evenly spread entries would put the
// target (the position's standard deviation is at most sqrt(entries) / 2), the
// later ones splitting what is left evenly.
__device__ uint64_t wave_lower_bound(const uint32_t* idx, uint64_t lo, uint64_t hi, uint64_t target,
                                     float x) {
  const int lane = lane_id();
  bool guess = true;
  while (hi - lo > 64) {
    const uint64_t span = hi - lo;  // < 2^58
    uint64_t at = lo + span * (uint64_t)((lane & 15) + 1) / 17u;
    if (guess) {
      // 16 distinct ascending positions in [lo, hi)
      guess = false;
      const float s = (float)span;
      const int64_t step = 1 + (int64_t)(__builtin_sqrtf(s) * 0.125f);
      int64_t q = (int64_t)(s * x) + ((lane & 15) - 8) * step;
      const int64_t bot = lane & 15, top = (int64_t)span - 16 + (lane & 15);
      q = q < bot ? bot : q > top ? top : q;
      at = lo + (uint64_t)q;
    }
    const uint32_t ge = (uint32_t)__ballot(lane < 16 && (uint64_t)idx[lane < 16 ? at : lo] >= target);
    if (ge == 0) {
      lo = __shfl(at, 15, 64) + 1;  // every probe is below the target
    } else {
      const int q = __builtin_ctz(ge);
      const uint64_t pb = q > 0 ? __shfl(at, q - 1, 64) + 1 : lo;
      hi = __shfl(at, q, 64);  // idx[hi] >= target: the answer is at most there
      lo = pb;
    }
  }
  const uint64_t k = lo + (uint64_t)lane;
  const uint64_t ge = __ballot(k < hi && (uint64_t)idx[k < hi ? k : lo] >= target);
  return ge == 0 ? hi : lo + (uint64_t)__builtin_ctzll(ge);
}

__device__ __forceinline__ float4 ld4(const float* p) {
  const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                     __uint_as_float(v.w));
}

__device__ __forceinline__ void st4(float* p, float4 v) {
  u32x4_t w;
  w.x = __float_as_uint(v.x);
  w.y = __float_as_uint(v.y);
  w.z = __float_as_uint(v.z);
  w.w = __float_as_uint(v.w);
  __builtin_nontemporal_store(w, reinterpret_cast<u32x4_t*>(p));
}

// The update of one element (each line one FP32 rounding).
__device__ __forceinline__ void nesterov(float& th, float& m, float g, float mu, float alpha) {
  float mm = mu * m;
  mm = mm + g;
  m = mm;
  float t = mu * mm;
  t = t + g;
  const float step = alpha * t;
  th = th - step;
}

// Tensor of a block-uniform tile: the last tensor whose first tile is <= tile
// (starts never decrease; an empty tensor shares its start with the next one,
// which wins).  A binary search with scalar loads of the kernel arguments.
__device__ __forceinline__ int outer_owner(const OuterParams& p, uint32_t tile) {
  static_assert(kMaxBatch == 64, "six halvings cover 64 tensors");
  uint32_t k = 0;
#pragma unroll
  for (uint32_t step = 32; step > 0; step >>= 1) {
    const uint32_t q = k + step;
    if (q < (uint32_t)p.ntensors && p.tile_begin[q] <= tile) k = q;
  }
  return (int)k;
}

}  // namespace

template <bool SMALL>
__global__ __launch_bounds__(kOuterTB) void outer_kernel(OuterParams p) {
  __shared__ float4 s_g[kOuterTile / 4];
  __shared__ uint64_t s_more[kMaxLists];  // entries of the tile past the held ones: from here
  __shared__ uint32_t s_cnt[kMaxLists];   // how many
  const int tid = threadIdx.x;
  const int wid = SMALL ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const int R = p.nlists;
  const int k = outer_owner(p, blockIdx.x);
  float* const theta = p.t[k].theta;
  float* const momentum = p.t[k].momentum;
  const uint64_t n = p.t[k].n;
  const uint32_t base = p.t[k].index_base;
  const uint64_t t0 = (uint64_t)(blockIdx.x - p.tile_begin[k]) * kOuterTile;
  const uint64_t t1 = t0 + kOuterTile < n ? t0 + kOuterTile : n;
  // this thread's elements: float4 j at t0 + (j * TB + tid) * 4, in flight
  // during the searches
  float4 th[kOuterVec], mo[kOuterVec];
  const bool full = t0 + kOuterTile <= n;
#pragma unroll
  for (int j = 0; j < kOuterVec; ++j) {
    const uint64_t e = t0 + (uint64_t)(j * kOuterTB + tid) * 4;
    if (full) {
      th[j] = ld4(theta + e);
      mo[j] = ld4(momentum + e);
    } else {
      float a[4], b[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        a[c] = e + c < t1 ? theta[e + c] : 0.0f;
        b[c] = e + c < t1 ? momentum[e + c] : 0.0f;
      }
      th[j] = make_float4(a[0], a[1], a[2], a[3]);
      mo[j] = make_float4(b[0], b[1], b[2], b[3]);
    }
    s_g[j * kOuterTB + tid] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
  // Wave r takes list r: it finds the list's first entry in the tile and holds
  // the entries from there on, kHeld per lane.
  const uint64_t lo_idx = (uint64_t)base + t0;
  const uint64_t hi_idx = (uint64_t)base + t1;  // <= index_base + n <= 2^32
  const int lane = lane_id();
  uint32_t id[kHeld];
  float v[kHeld];
#pragma unroll
  for (int h = 0; h < kHeld; ++h) {
    id[h] = 0xFFFFFFFFu;  // with v = 0: no entry
    v[h] = 0.0f;
  }
  if (wid < R) {
    const OuterListDesc& L = p.l[wid];
    const uint64_t cap = L.capacity;
    uint64_t lo = L.seg_begin[k];
    uint64_t hi = k + 1 < p.ntensors ? L.seg_begin[k + 1] : *L.end;
    lo = lo < cap ? lo : cap;
    hi = hi < cap ? hi : cap;
    hi = hi > lo ? hi : lo;
    const bool first = SMALL && t0 == 0;
    uint64_t f = lo;
    auto find = [&] { f = wave_lower_bound(L.idx, lo, hi, lo_idx, (float)t0 / (float)n); };
    if (!first) find();
    auto hold = [&](int h) {
      const uint64_t at = f + (uint64_t)(h * 64 + lane);
      if (at < hi) {
        id[h] = L.idx[at];
        v[h] = L.val[at];
      }
    };
    // whether the list goes on in the tile past the first h entries per lane
    auto goes_on = [&](int h) {
      return __ballot(lane == 63 && f + (uint64_t)(h * 64) < hi && (uint64_t)id[h - 1] < hi_idx) != 0;
    };
#pragma unroll
    for (int h = 0; h < kFirst; ++h) hold(h);
    if (first && __ballot(lane == 0 && lo < hi && (uint64_t)id[0] < lo_idx) != 0) {
      find();  // past entries below the tensor, which are ignored
#pragma unroll
      for (int h = 0; h < kFirst; ++h) {
        id[h] = 0xFFFFFFFFu;
        v[h] = 0.0f;
        hold(h);
      }
    }
    uint64_t m0 = f + kHeld * 64, m1 = m0;  // entries that are not held: dense lists
    if (goes_on(kFirst)) {
#pragma unroll
      for (int h = kFirst; h < kHeld; ++h) hold(h);
      if (goes_on(kHeld)) {
        // ascending distinct indices: at most a tile's elements (which also
        // bounds the work for a list out of order)
        const uint64_t top = f + kOuterTile < hi ? f + kOuterTile : hi;
        m1 = wave_lower_bound(L.idx, m0, top, hi_idx, (float)(t1 - t0) / (float)kOuterTile);
      }
    }
    if (lane == 0) {
      s_more[wid] = m0;
      s_cnt[wid] = (uint32_t)(m1 - m0);
    }
  }
  __syncthreads();  // g is zero everywhere
  // Scatter-add, worker by worker: the entries of one list are distinct, so
  // its adds never collide, and a barrier orders the workers.
  float* g = reinterpret_cast<float*>(s_g);
  for (int r = 0; r < R; ++r) {
    if (r == wid) {
#pragma unroll
      for (int h = 0; h < kHeld; ++h) {
        const uint64_t o = (uint64_t)id[h] - lo_idx;
        if (o < t1 - t0 && (id[h] != 0xFFFFFFFFu || v[h] != 0.0f)) g[o] += v[h];
      }
    }
    const uint32_t more = s_cnt[r];
    for (uint32_t c = (uint32_t)tid; c < more; c += kOuterTB) {
      const uint64_t o = (uint64_t)p.l[r].idx[s_more[r] + c] - lo_idx;
      if (o < t1 - t0) g[o] += p.l[r].val[s_more[r] + c];
    }
    __syncthreads();
  }
  // R a power of two: the product by 1 / R rounds to the same value as the quotient
  const float rf = (float)R;
  const bool pow2 = (R & (R - 1)) == 0;
  const float inv = R > 0 ? 1.0f / rf : 1.0f;
#pragma unroll
  for (int j = 0; j < kOuterVec; ++j) {
    const uint64_t e = t0 + (uint64_t)(j * kOuterTB + tid) * 4;
    float4 gv = s_g[j * kOuterTB + tid];
    if (pow2) {
      gv.x = gv.x * inv;
      gv.y = gv.y * inv;
      gv.z = gv.z * inv;
      gv.w = gv.w * inv;
    } else {
      gv.x = gv.x / rf;
      gv.y = gv.y / rf;
      gv.z = gv.z / rf;
      gv.w = gv.w / rf;
    }
    nesterov(th[j].x, mo[j].x, gv.x, p.mu, p.alpha);
    nesterov(th[j].y, mo[j].y, gv.y, p.mu, p.alpha);
    nesterov(th[j].z, mo[j].z, gv.z, p.mu, p.alpha);
    nesterov(th[j].w, mo[j].w, gv.w, p.mu, p.alpha);
    if (full) {
      st4(theta + e, th[j]);
      st4(momentum + e, mo[j]);
    } else {
      const float a[4] = {th[j].x, th[j].y, th[j].z, th[j].w};
      const float b[4] = {mo[j].x, mo[j].y, mo[j].z, mo[j].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (e + c < t1) {
          theta[e + c] = a[c];
          momentum[e + c] = b[c];
        }
      }
    }
  }
}

uint64_t outer_tile_elems() { return kOuterTile; }
uint64_t outer_max_tiles() { return 0xFFFFFFFFull / kOuterTB; }

hipError_t launch_outer(const OuterParams& p, hipStream_t stream) {
  if (p.ntiles == 0) return hipSuccess;
  if (p.ntiles <= kSmallTiles)
    hipLaunchKernelGGL(outer_kernel<true>, dim3(p.ntiles), dim3(kOuterTB), 0, stream, p);
  else
    hipLaunchKernelGGL(outer_kernel<false>, dim3(p.ntiles), dim3(kOuterTB), 0, stream, p);
  return hipGetLastError();
}

}  // namespace pulse
