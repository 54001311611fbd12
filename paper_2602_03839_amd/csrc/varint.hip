// varint.hip -- the encoders of a sorted patch's two index streams on gfx950:
//
//   * the delta-varint stream (App. H.2 "Index Encoding": first index as it
//     is, then differences; App. F.3 "Sparse stream format": delta-encoded,
//     varint-packed indices).  Each number is an unsigned varint: 7-bit
//     groups, least significant first, every byte but the last carrying 0x80.
//     A patch of several tensors is a list of segments (one per tensor);
//     every segment restarts with its first index as it is.
//   * the 2-D COO delta downcast of App. H.2 step 4 / App. H.4.1: per tensor
//     (row-major, `cols` columns) the first index as it is, then one (uint8 row
//     field, uint16 column field) pair per later entry -- (0, column gap)
//     within a row, (rows ahead, column + 1) on a later row -- with (255, 0)
//     escape pairs, each 255 rows, ahead of a gap of more than 255 rows.
//
// Both place each entry's output by an exclusive sum of per-entry sizes (its
// varint length, or its pair count: 1 + its escapes, 0 for a segment's first
// entry), computed reduce-then-write over tiles of entries (stream_common.hpp):
// a size pass per tile, and an emit pass that recomputes the sizes and writes
// the unit's output as one contiguous run.  The decoders are in decode.hip.
//
// A thread takes four quads of consecutive entries straight from memory; the
// entry before a quad comes from the lane before.  A unit without a segment
// start (nearly all of a large patch's) passes two barriers in the varint emit
// pass and one in the COO's, whose pairs then lie where their entries do.
// Measured against staging every entry in LDS and writing single bytes: 7B
// set's patch (71M entries, 255 segments), varint size and emit 92 + 223 ->
// 85 + 120 us; 0.5B set's (4.6M, 218), COO 20 + 44 -> 10 + 33 us, and no
// launch between the passes (8 and 5 us).  The size pass is bound by reading
// the list (285 MB at 3.3 TB/s while the caches write back what the call
// before wrote); the emit passes by instruction issue and occupancy.
#include "launch.hpp"
#include "stream_common.hpp"

namespace pulse {

using namespace stream;

namespace {

constexpr uint32_t kStageBytes = 3 * kDUnit;  // bytes of a unit staged in LDS

__device__ __forceinline__ uint32_t varint_len(uint32_t d) {
  return d < (1u << 7) ? 1u : d < (1u << 14) ? 2u : d < (1u << 21) ? 3u : d < (1u << 28) ? 4u : 5u;
}

struct Tile {
  uint64_t nent, t0, t1;
  bool some;  // this block has a tile
  bool last;
  uint32_t ntiles;
};

// This block's tile of the entries below min(*end, capacity).
__device__ __forceinline__ Tile entry_tile(const uint64_t* end, uint64_t capacity) {
  Tile t;
  const uint64_t e = *end;
  t.nent = e < capacity ? e : capacity;
  const Geo g = stream_geometry(t.nent);
  t.some = blockIdx.x < g.ntiles;
  t.last = blockIdx.x + 1 == g.ntiles;
  t.ntiles = g.ntiles;
  t.t0 = (uint64_t)blockIdx.x * g.tile;
  t.t1 = t.t0 + g.tile < t.nent ? t.t0 + g.tile : t.nent;
  return t;
}

// A tensor's column count C with its reciprocal, for row = index / C.
struct Cols {
  uint32_t C;
  double rc;  // 1 / C, rounded
};

__device__ __forceinline__ Cols make_cols(uint32_t c) {
  Cols k;
  k.C = c > 0 ? c : 1u;
  k.rc = 1.0 / (double)k.C;
  return k;
}

// floor(x / C).  x * rc is within 2^-20 of x / C (x < 2^32, both roundings
// relative 2^-53), so its truncation is the quotient or one off, which the
// remainder check corrects; no integer division (a long instruction sequence
// on the GPU) per entry.
__device__ __forceinline__ uint32_t div_cols(uint32_t x, const Cols& k) {
  uint32_t q = (uint32_t)((double)x * k.rc);
  const uint64_t qc = (uint64_t)q * k.C;
  if (qc > x) --q;
  else if (x - (uint32_t)qc >= k.C) ++q;
  return q;
}

// A walk over a thread's entries of one tensor: the row and column of the last.
struct CooAt {
  uint32_t prev, col;
};

// The 2-D COO pairs of entry cur after the walk's last entry: the last pair (row
// field << 16 | column field) in *last, and their number.  The columns between
// two entries decide: less than a row apart, the next row is at most one away,
// and no division is needed.
__device__ __forceinline__ uint32_t coo_step(CooAt& at, uint32_t cur, const Cols& k, uint32_t* last) {
  const uint32_t gap = cur - at.prev;
  uint32_t np = 1;
  if (gap < k.C) {
    const uint32_t c = at.col + gap;
    const bool next = c >= k.C;
    *last = next ? (1u << 16) | (c - k.C + 1) : gap;
    at.col = next ? c - k.C : c;
  } else {
    const uint32_t r = div_cols(cur, k), pr = div_cols(at.prev, k);
    at.col = cur - r * k.C;
    const uint32_t dr = r - pr;
    if (cur < at.prev) {  // not ascending (outside the contract): one pair, no escapes
      *last = 0;
    } else {
      const uint32_t esc = (dr - 1) / 255u;
      *last = ((dr - 255u * esc) << 16) | (at.col + 1);
      np += esc;
    }
  }
  at.prev = cur;
  return np;
}

// The segment of entry k of a tile (its cached starts C): the last one starting
// at or before it (0 if none).
__device__ __forceinline__ uint32_t segment_at(const uint64_t* starts, const SegCache& C, uint64_t k) {
  return segment_of(starts, C, C.lo, C.lo + C.n, k);
}

}  // namespace

// ---------------------------------------------------------------- delta-varint
//
// Table word b: tile b's byte count.

__global__ __launch_bounds__(kDT) void varint_size_kernel(VarintEncParams p) {
  __shared__ uint32_t s_bits[kDUnit / 32];
  __shared__ uint32_t s_w[kDWaves];
  __shared__ SegCache s_seg;
  const Tile t = entry_tile(p.end, p.capacity);
  if (!t.some) return;
  Quads x = load_quads(p.idx, t.t0, t.t1);
  cache_tile_segments(p.seg_begin, p.nseg, t.t0, t.t1, s_seg);
  uint32_t bytes = 0;  // < 5 * tile
  for (uint64_t u0 = t.t0; u0 < t.t1; u0 += kDUnit) {
    const uint64_t u1 = u0 + kDUnit < t.t1 ? u0 + kDUnit : t.t1;
    Quads cur = x;
    x = load_quads(p.idx, u1, u1 + kDUnit < t.t1 ? u1 + kDUnit : t.t1);  // in flight (zeros past the tile)
    finish_quads(cur, p.idx, u0, u1);
    mark_unit(p.seg_begin, s_seg, u0, u1, s_bits);
    const uint32_t marks = quad_marks(s_seg, s_bits);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t before = before_quad(cur, q), m = quad_len(u0, u1, q);
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t i = 4 * q + j;
        const uint32_t d = cur.v[i] - ((marks >> i) & 1u ? 0u : j ? cur.v[i - 1] : before);
        bytes += j < m ? varint_len(d) : 0u;
      }
    }
    if (s_seg.n) __syncthreads();  // the bitmap is rewritten by the next unit
  }
  uint32_t total;
  (void)block_count_excl(bytes, s_w, &total);
  if (threadIdx.x == 0) stream_words(p.ws)[blockIdx.x] = total;
}

__global__ __launch_bounds__(kDT) void varint_emit_kernel(VarintEncParams p) {
  __shared__ uint32_t s_bits[kDUnit / 32];
  __shared__ uint2 s_w[2][kDWaves];
  __shared__ uint64_t s_w64[kDWaves];
  __shared__ SegCache s_seg;
  __shared__ uint32_t s_quad[kDUnit / 4];
  __shared__ __align__(16) uint8_t s_bytes[2][kStageBytes + 32];
  static_assert(5 * kDUnit < 1u << 15, "a unit's byte offsets fit 15 bits");
  const int tid = (int)threadIdx.x;
  const Tile t = entry_tile(p.end, p.capacity);
  if (!t.some) return;
  Quads x = load_quads(p.idx, t.t0, t.t1);
  uint64_t base = fold_before(stream_words(p.ws), blockIdx.x, s_w64);
  cache_tile_segments(p.seg_begin, p.nseg, t.t0, t.t1, s_seg);
  int buf = 0;
  for (uint64_t u0 = t.t0; u0 < t.t1; u0 += kDUnit, buf ^= 1) {
    const uint64_t u1 = u0 + kDUnit < t.t1 ? u0 + kDUnit : t.t1;
    Quads cur = x;
    x = load_quads(p.idx, u1, u1 + kDUnit < t.t1 ? u1 + kDUnit : t.t1);  // in flight (zeros past the tile)
    finish_quads(cur, p.idx, u0, u1);
    mark_unit(p.seg_begin, s_seg, u0, u1, s_bits);
    const uint32_t marks = quad_marks(s_seg, s_bits);
    uint32_t d[16], m[4], size[4], at[4], ubytes, top = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t before = before_quad(cur, q);
      m[q] = quad_len(u0, u1, q);
      size[q] = 0;
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t i = 4 * q + j;
        d[i] = cur.v[i] - ((marks >> i) & 1u ? 0u : j ? cur.v[i - 1] : before);
        if (j >= m[q]) d[i] = 0;
        size[q] += j < m[q] ? varint_len(d[i]) : 0u;
        top |= d[i];
      }
    }
    scan_quads(size, s_w, buf, at, &ubytes);
    // The unit's bytes are one contiguous run [base, base + ubytes).  Up to
    // kStageBytes of them (always, below ~3 bytes per index) are staged, at
    // the alignment they have in memory, and written in aligned 16-byte
    // chunks; a longer run is written by each thread for its own entries.
    const bool staged = ubytes <= kStageBytes;  // block-uniform
    const uint32_t sh = (uint32_t)((uintptr_t)(p.out + base) & 15u);
    if (staged) {
      uint8_t* const to = s_bytes[buf] + sh;
      if (__ballot(top >= (1u << 14)) == 0) {
        // one or two bytes each
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t o = at[q];
#pragma unroll
          for (uint32_t j = 0; j < 4; ++j) {
            const uint32_t v = d[4 * q + j];
            if (j < m[q]) {
              const bool two = v >= 128u;
              to[o] = (uint8_t)((v & 0x7Fu) | (two ? 0x80u : 0u));
              if (two) to[o + 1] = (uint8_t)(v >> 7);
              o += two ? 2u : 1u;
            }
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint32_t o = at[q];
#pragma unroll
          for (uint32_t j = 0; j < 4; ++j) {
            uint32_t v = d[4 * q + j];
            if (j < m[q]) {
              const uint32_t len = varint_len(v);
              for (uint32_t b = 0; b < len; ++b) {
                to[o + b] = (uint8_t)((v & 0x7Fu) | (b + 1 < len ? 0x80u : 0u));
                v >>= 7;
              }
              o += len;
            }
          }
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint64_t o = base + at[q];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
          uint32_t v = d[4 * q + j];
          if (j < m[q]) {
            const uint32_t len = varint_len(v);
            for (uint32_t b = 0; b < len; ++b) {
              if (o + b < p.out_capacity) p.out[o + b] = (uint8_t)((v & 0x7Fu) | (b + 1 < len ? 0x80u : 0u));
              v >>= 7;
            }
            o += len;
          }
        }
      }
    }
    // per quad, for the segments that start in the unit: the quad's first byte,
    // and the bytes of its first one, two and three entries (15 + 3 x 4 bits)
    const bool starts = s_seg.n != 0 && p.seg_bytes;  // block-uniform
    if (starts) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t w = at[q], o = 0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          o += varint_len(d[4 * q + j]);
          w |= o << (15 + 4 * j);
        }
        s_quad[q * kDT + tid] = w;
      }
    }
    __syncthreads();
    // A lane per segment (the thread that holds a segment's first entry, walking
    // its sixteen, made the wave wait for up to sixteen searches: a 300K set's
    // patch in 300 tensors 30.4 -> 12.9 us).
    if (starts) {
      for (uint32_t i = (uint32_t)tid; i < s_seg.n; i += kDT) {
        const uint32_t s = s_seg.lo + i;
        const uint64_t v = start_of(p.seg_begin, s_seg, s);
        if (v >= u0 && v < u1) {
          const uint32_t e = (uint32_t)(v - u0), w = s_quad[e >> 2];
          p.seg_bytes[s] = base + (w & 0x7FFFu) + ((e & 3u) ? (w >> (11u + 4u * (e & 3u))) & 0xFu : 0u);
        }
      }
    }
    if (staged) {
      const uint8_t* const from = s_bytes[buf];
      for (uint32_t c = (uint32_t)tid * 16; c < sh + ubytes; c += kDT * 16) {
        const uint64_t g = base + c - sh;  // of the chunk's first byte (may lie before the unit)
        if (c >= sh && c + 16 <= sh + ubytes && g + 16 <= p.out_capacity) {
          *reinterpret_cast<uint4*>(p.out + g) = *reinterpret_cast<const uint4*>(from + c);
        } else {
          for (uint32_t b = c < sh ? sh : c; b < c + 16 && b < sh + ubytes; ++b)
            if (base + (b - sh) < p.out_capacity) p.out[base + (b - sh)] = from[b];
        }
      }
    }
    base += ubytes;
    // no barrier here: the next unit stages into the other buffer, and its
    // scan's barrier separates this unit's copy from the unit after it
  }
  if (t.last) {
    // the stream's length, and the segments that start at or past the last entry
    if (tid == 0) *p.total = base;
    if (p.seg_bytes && p.nseg > 0 && tid < 64) {
      const uint32_t from = lower_bound_wave(p.seg_begin, p.nseg, t.nent);
      for (uint32_t s = from + (uint32_t)lane_id(); s < p.nseg; s += 64) p.seg_bytes[s] = base;
    }
  }
  stream_finish(p.ws, t.ntiles, t.ntiles);
}

// ---------------------------------------------------------------- 2-D COO
//
// Table word b: tile b's pair count.

__device__ __forceinline__ Cols cols_at(const CooEncParams& p, const SegCache& C, uint64_t k) {
  return make_cols(p.cols[segment_at(p.seg_begin, C, k)]);
}

__global__ __launch_bounds__(kDT) void coo_size_kernel(CooEncParams p) {
  __shared__ uint32_t s_bits[kDUnit / 32];
  __shared__ uint64_t s_w[kDWaves];
  __shared__ SegCache s_seg;
  const Tile t = entry_tile(p.end, p.capacity);
  if (!t.some) return;
  Quads x = load_quads(p.idx, t.t0, t.t1);
  cache_tile_segments(p.seg_begin, p.nseg, t.t0, t.t1, s_seg);
  const uint32_t c_first = p.cols[segment_at(p.seg_begin, s_seg, t.t0)];
  uint64_t pairs = 0;
  for (uint64_t u0 = t.t0; u0 < t.t1; u0 += kDUnit) {
    const uint64_t u1 = u0 + kDUnit < t.t1 ? u0 + kDUnit : t.t1;
    Quads cur = x;
    x = load_quads(p.idx, u1, u1 + kDUnit < t.t1 ? u1 + kDUnit : t.t1);  // in flight (zeros past the tile)
    finish_quads(cur, p.idx, u0, u1);
    mark_unit(p.seg_begin, s_seg, u0, u1, s_bits);
    const uint32_t marks = quad_marks(s_seg, s_bits);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint64_t k = u0 + 4ull * ((uint32_t)q * kDT + threadIdx.x);
      const uint32_t before = before_quad(cur, q), m = quad_len(u0, u1, q);
      uint32_t C = c_first;
      if (s_seg.n && m) C = p.cols[segment_at(p.seg_begin, s_seg, k)];
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t i = 4 * q + j;
        if (j < m) {
          const uint32_t prev = j ? cur.v[i - 1] : before, v = cur.v[i];
          if ((marks >> i) & 1u || k + j == 0) {
            // a segment's first entry has no pair
            if (j) C = p.cols[segment_at(p.seg_begin, s_seg, k + j)];
          } else {
            const uint32_t c = C > 0 ? C : 1u;
            ++pairs;
            // entries fewer than 255 rows apart have no escape, whatever their columns
            if ((uint64_t)(v - prev) >= 255ull * c && v >= prev) pairs += (v / c - prev / c - 1) / 255u;
          }
        }
      }
    }
    if (s_seg.n) __syncthreads();  // the bitmap is rewritten by the next unit
  }
  // block sum (64-bit: escapes may be many)
  const uint64_t w = wave_sum_u64(pairs);
  if (lane_id() == 0) s_w[threadIdx.x >> 6] = w;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t total = 0;
    for (int v = 0; v < kDWaves; ++v) total += s_w[v];
    stream_words(p.ws)[blockIdx.x] = total;
  }
}

// Four or eight bytes at any address (the compiler stores them as the target
// takes them, from the declared alignment of 1).
typedef uint32_t u32_a1 __attribute__((aligned(1)));
typedef uint32_t u32x2_a1 __attribute__((ext_vector_type(2), aligned(1)));

__global__ __launch_bounds__(kDT) void coo_emit_kernel(CooEncParams p) {
  __shared__ uint32_t s_bits[kDUnit / 32];
  __shared__ SegCache s_seg;
  __shared__ uint32_t s_ent[padded(kDUnit + 1)];    // at pad(0) the entry before the unit, at pad(1 + i) entry i
  __shared__ uint32_t s_pairs[padded(kDUnit + 1)];  // the unit's pairs, pair q at pad(q)
  __shared__ Sum64 s_w64[kDWaves];
  __shared__ uint64_t s_wf[kDWaves];
  const int tid = (int)threadIdx.x;
  const Tile t = entry_tile(p.end, p.capacity);
  if (!t.some) return;
  Quads x = load_quads(p.idx, t.t0, t.t1);
  uint64_t base = fold_before(stream_words(p.ws), blockIdx.x, s_wf);
  cache_tile_segments(p.seg_begin, p.nseg, t.t0, t.t1, s_seg);
  const Cols c_first = cols_at(p, s_seg, t.t0);
  for (uint64_t u0 = t.t0; u0 < t.t1; u0 += kDUnit) {
    const uint64_t u1 = u0 + kDUnit < t.t1 ? u0 + kDUnit : t.t1;
    Quads cur = x;
    x = load_quads(p.idx, u1, u1 + kDUnit < t.t1 ? u1 + kDUnit : t.t1);  // in flight (zeros past the tile)
    finish_quads(cur, p.idx, u0, u1);
    mark_unit(p.seg_begin, s_seg, u0, u1, s_bits);
    // A unit of one segment whose entries lie fewer than 255 rows apart has one
    // pair for each: they lie where the entries do, and if all of them fit the
    // buffer they are written at once.
    bool one = s_seg.n == 0 && u0 > 0;
    const uint64_t far = 255ull * c_first.C;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t before = before_quad(cur, q), m = quad_len(u0, u1, q);
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t gap = cur.v[4 * q + j] - (j ? cur.v[4 * q + j - 1] : before);
        one &= j >= m || (uint64_t)gap < far;
      }
    }
    if (__syncthreads_and(one) && base + (u1 - u0) <= p.out_capacity) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint64_t g = base + 4ull * ((uint32_t)q * kDT + (uint32_t)tid);
        const uint32_t m = quad_len(u0, u1, q), before = before_quad(cur, q);
        CooAt at{before, before - div_cols(before, c_first) * c_first.C};
        uint32_t l[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
          l[j] = 0;
          if (j < m) (void)coo_step(at, cur.v[4 * q + j], c_first, &l[j]);
        }
        if (m == 4) {
          *reinterpret_cast<u32_a1*>(p.drow + g) =
              (l[0] >> 16) | ((l[1] >> 16) << 8) | ((l[2] >> 16) << 16) | ((l[3] >> 16) << 24);
          *reinterpret_cast<u32x2_a1*>(p.dcol + g) =
              u32x2_a1{(l[0] & 0xFFFFu) | (l[1] << 16), (l[2] & 0xFFFFu) | (l[3] << 16)};
        } else {
#pragma unroll
          for (uint32_t j = 0; j < 3; ++j) {
            if (j < m) {
              p.drow[g + j] = (uint8_t)(l[j] >> 16);
              p.dcol[g + j] = (uint16_t)l[j];
            }
          }
        }
      }
      base += u1 - u0;
      continue;
    }
    // The general unit: its entries go through LDS, a thread takes sixteen
    // consecutive ones in loops that are not unrolled (unrolled, this path's
    // registers left two waves per SIMD to the one above: 41 us instead of 33
    // for the 0.5B set's patch).
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t i = 4u * ((uint32_t)q * kDT + (uint32_t)tid);
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) s_ent[pad(1 + i + j)] = cur.v[4 * q + j];
    }
    if (tid == 0) s_ent[pad(0)] = cur.edge[0];
    __syncthreads();
    const uint32_t run = run_marks(s_seg, s_bits);
    const uint32_t i0 = 16u * (uint32_t)tid;
    const uint64_t k0 = u0 + i0;
    const uint32_t m = k0 < u1 ? (uint32_t)(u1 - k0 < 16 ? u1 - k0 : 16) : 0u;
    // f(entry, its last pair, its pairs: one and its escapes, none for a
    // segment's first entry)
    auto walk = [&](auto f) {
      Cols c = c_first;
      if (s_seg.n && m) c = cols_at(p, s_seg, k0);
      const uint32_t before = s_ent[pad(i0)];
      CooAt at{before, before - div_cols(before, c) * c.C};
#pragma unroll 1
      for (uint32_t j = 0; j < m; ++j) {
        const uint32_t v = s_ent[pad(1 + i0 + j)];
        uint32_t last = 0, np = 0;
        if ((run >> j) & 1u || k0 + j == 0) {
          if (j) c = cols_at(p, s_seg, k0 + j);
          at.prev = v;
          at.col = v - div_cols(v, c) * c.C;
        } else {
          np = coo_step(at, v, c, &last);
        }
        f(j, v, last, np);
      }
    };
    uint64_t sum = 0;
    walk([&](uint32_t, uint32_t, uint32_t, uint32_t np) { sum += np; });
    // 64-bit offsets: valid lists keep a unit's pairs far below 2^32, but an
    // unsorted one need not, and positions must stay exact for the bounds
    // checks below to bound the work
    Sum64 all;
    uint64_t at = block_scan_excl<kDT>(Sum64{sum}, Sum64::id(), s_w64, &all).v;
    const uint64_t upairs = all.v;
    // Without long escapes the unit's pairs fit s_pairs (as row field << 16 |
    // column field) and consecutive lanes write consecutive pairs; otherwise
    // each thread writes its own entries' pairs, stopping at the output
    // capacity, so the work stays bounded by the buffer even for a list
    // outside the contract.
    const bool staged = upairs <= kDUnit + 1;
    walk([&](uint32_t j, uint32_t v, uint32_t l, uint32_t n) {
      // segments starting here: their pair offset and first index, from the
      // thread that holds their first entry
      if ((run >> j) & 1u) {
        for (uint32_t s = lower_bound_cached(p.seg_begin, s_seg, k0 + j);
             s < s_seg.lo + s_seg.n && start_of(p.seg_begin, s_seg, s) == k0 + j; ++s) {
          const uint64_t e = s + 1 < p.nseg ? p.seg_begin[s + 1] : t.nent;
          p.seg_pairs[s] = base + at;
          p.first[s] = e > k0 + j ? v : 0u;
        }
      }
      if (staged) {
        for (uint32_t r = 0; r + 1 < n; ++r) s_pairs[pad((uint32_t)at + r)] = 255u << 16;
        if (n) s_pairs[pad((uint32_t)at + n - 1)] = l;
      } else {
        for (uint32_t r = 0; r < n && base + at + r < p.out_capacity; ++r) {
          p.drow[base + at + r] = (uint8_t)(r + 1 < n ? 255u : l >> 16);
          p.dcol[base + at + r] = (uint16_t)(r + 1 < n ? 0u : l);
        }
      }
      at += n;
    });
    __syncthreads();
    if (staged) {
      for (uint32_t q = (uint32_t)tid; q < (uint32_t)upairs; q += kDT) {
        const uint64_t g = base + q;
        if (g < p.out_capacity) {
          const uint32_t pair = s_pairs[pad(q)];
          p.drow[g] = (uint8_t)(pair >> 16);
          p.dcol[g] = (uint16_t)(pair & 0xFFFFu);
        }
      }
    }
    __syncthreads();  // s_ent, s_pairs and the bitmap are rewritten by a later unit
    base += upairs;
  }
  if (t.last) {
    // the stream's length, and the pair offset (and first index 0) of every
    // segment that starts at or past the last entry
    if (tid == 0) *p.total = base;
    if (tid < 64) {
      const uint32_t from = lower_bound_wave(p.seg_begin, p.nseg, t.nent);
      for (uint32_t s = from + (uint32_t)lane_id(); s < p.nseg; s += 64) {
        p.seg_pairs[s] = base;
        p.first[s] = 0u;
      }
    }
  }
  stream_finish(p.ws, t.ntiles, t.ntiles);
}

hipError_t launch_varint_encode(const VarintEncParams& p, hipStream_t stream) {
  const uint32_t grid = tile_grid(p.capacity);
  hipLaunchKernelGGL(varint_size_kernel, dim3(grid), dim3(kDT), 0, stream, p);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(varint_emit_kernel, dim3(grid), dim3(kDT), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_coo_encode(const CooEncParams& p, hipStream_t stream) {
  const uint32_t grid = tile_grid(p.capacity);
  hipLaunchKernelGGL(coo_size_kernel, dim3(grid), dim3(kDT), 0, stream, p);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(coo_emit_kernel, dim3(grid), dim3(kDT), 0, stream, p);
  return hipGetLastError();
}

}  // namespace pulse
