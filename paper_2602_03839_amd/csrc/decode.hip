// decode.hip -- the decoders of the patch's two index streams on gfx950, Alg. 1
// Decode's DeltaDecode (and Upcast) steps for
//   * the delta-varint stream (App. H.2 "Index Encoding", App. F.3 "Sparse
//     stream format"): per segment the first index as it is, then differences,
//     each an unsigned LEB128 varint;
//   * the 2-D COO delta downcast (App. H.2 step 4, App. H.4.1 "Type
//     downscaling"): per segment the first index, then (uint8 row field,
//     uint16 column field) pairs, with (255, 0) escapes for long row gaps.
//
// Both decodes are running sums: an entry's index sums the differences since
// its segment's start, and its place counts the numbers (or non-escape pairs)
// before it.  Each is computed reduce-then-write over tiles of the stream
// (stream_common.hpp), so that no block ever waits on another:
//   * COO: a reduce pass folds each tile's pairs into one map on (row,
//     column, escapes), one block composes the maps, and a write pass gives
//     every pair its entry's index and place;
//   * delta-varint: a count pass (terminating bytes, plain sum of the
//     numbers); a pass with one block per segment that gives the tiles whose
//     first entry lies in it that entry and the sum carried into it (the plain
//     sum before the tile less the one before the segment); and a write pass.
// The indices are written once, staged in LDS so that consecutive lanes store
// consecutive entries.  (The single-pass form with a decoupled look-back per
// tile was bound by the look-back latency: 3.3 and 5.7 ms on a 306M-entry
// patch.)
#include "launch.hpp"
#include "stream_common.hpp"

namespace pulse {

using namespace stream;

namespace {

// Segmented sum: f = a restart (a segment start) occurred, s = the sum since
// the last one (or since the start, with no restart).
struct SegSum {
  uint32_t f, s;
  __device__ static SegSum id() { return SegSum{0u, 0u}; }
};
__device__ __forceinline__ SegSum comb(SegSum x, SegSum y) {
  return SegSum{x.f | y.f, y.f ? y.s : x.s + y.s};
}
__device__ __forceinline__ SegSum shfl_up(SegSum x, int d) {
  return SegSum{(uint32_t)__shfl_up((int)x.f, d, 64), (uint32_t)__shfl_up((int)x.s, d, 64)};
}

// COO state.  Absolute (abs = 1): the current entry's row and column within
// its tensor, and the escapes since its segment's start.  Relative (abs = 0):
// the map a run of pairs applies to an absolute state --
//   row += a;  col = k ? col + b : b;  e += e
// -- which is how every pair acts: a same-row pair (0, gap) is (k 1, a 0,
// b gap), a pair dr rows down (dr, col + 1) is (k 0, a dr, b col), an escape
// (255, 0) is (k 1, a 255, b 0, e 1).  A segment start makes the state
// absolute again from the segment's first index.  Composition: k = k1 k2,
// a = a1 + a2, b = k2 ? b1 + b2 : b2, e = e1 + e2.
struct CooEl {
  uint32_t abs, k, a, b, e;
  __device__ static CooEl id() { return CooEl{0u, 1u, 0u, 0u, 0u}; }
};
__device__ __forceinline__ CooEl comb(CooEl x, CooEl y) {
  if (y.abs) return y;
  CooEl r;
  r.abs = x.abs;
  r.k = x.abs ? 1u : (x.k & y.k);
  r.a = x.a + y.a;
  r.b = y.k ? x.b + y.b : y.b;
  r.e = x.e + y.e;
  return r;
}
__device__ __forceinline__ CooEl shfl_up(CooEl x, int d) {
  CooEl r;
  r.abs = (uint32_t)__shfl_up((int)x.abs, d, 64);
  r.k = (uint32_t)__shfl_up((int)x.k, d, 64);
  r.a = (uint32_t)__shfl_up((int)x.a, d, 64);
  r.b = (uint32_t)__shfl_up((int)x.b, d, 64);
  r.e = (uint32_t)__shfl_up((int)x.e, d, 64);
  return r;
}

// ---------------------------------------------------------------- varint bytes

// Sixteen stream bytes [pos, pos + 16) of a thread (pos a multiple of 16, the
// stream 16-byte aligned) and the four before them.  Bytes before the stream
// read as 0 (a terminator: the first number starts at byte 0); bytes at or past
// n read as 0x80 (a continuation: a number cut by the end has no terminator
// and is dropped).
struct Bytes16 {
  uint32_t h;      // bytes pos - 4 .. pos - 1, the first in the low byte
  uint32_t w[4];   // bytes pos .. pos + 15
};

// This thread's sixteen bytes of the unit starting at u0 (none past u1; see
// "Prefetches" in stream_common.hpp).
__device__ __forceinline__ Bytes16 unit_bytes(const uint8_t* in, uint64_t u0, uint64_t u1) {
  const uint64_t pos = u0 + 16ull * threadIdx.x;
  const uint8_t* const zero = reinterpret_cast<const uint8_t*>(kStreamZero);
  const uint4 v = load16(pos + 16 <= u1 ? in + pos : zero);
  Bytes16 b;
  b.h = *reinterpret_cast<const uint32_t*>(pos >= 4 && pos < u1 ? in + pos - 4 : zero);
  b.w[0] = v.x;
  b.w[1] = v.y;
  b.w[2] = v.z;
  b.w[3] = v.w;
  return b;
}

// Sets the bytes of [u0, u1) that unit_bytes did not load: the ragged sixteen at
// the stream's end, and continuations (no terminators) past it.
__device__ __forceinline__ void finish_bytes(Bytes16& b, const uint8_t* in, uint64_t u0, uint64_t u1) {
  if (u0 + kDUnit <= u1) return;  // block-uniform
  const uint64_t pos = u0 + 16ull * threadIdx.x;
  if (pos + 16 <= u1) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t x = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint64_t at = pos + (uint64_t)(4 * q + c);
      const uint32_t byte = at < u1 ? (uint32_t)in[at] : 0x80u;
      x |= byte << (8 * c);
    }
    b.w[q] = x;
  }
}

__device__ __forceinline__ uint32_t terminators(const Bytes16& b) {
  uint32_t c = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) c += (uint32_t)__builtin_popcount(~b.w[q] & 0x80808080u);
  return c;
}

// Calls emit(value) for every number that ends in the sixteen bytes, in
// order.  A number starts after a terminator; it ends at most four bytes
// after its start in a valid stream, so starting the walk four bytes early
// finds the start of every number that ends in the sixteen.  (A number of
// more than five bytes is not a uint32 varint; its value is unspecified.)
template <typename Emit>
__device__ __forceinline__ void walk_numbers(const Bytes16& b, Emit emit) {
  uint32_t cur = 0, sh = 0;
  bool start = true;
#pragma unroll
  for (int j = -4; j < 16; ++j) {
    const uint32_t byte = j < 0 ? (b.h >> (8 * (j + 4))) & 0xFFu : (b.w[j >> 2] >> (8 * (j & 3))) & 0xFFu;
    const uint32_t v7 = byte & 0x7Fu;
    if (start) {
      cur = v7;
      sh = 7;
    } else {
      cur |= sh < 32 ? v7 << sh : 0u;
      sh += 7;
    }
    start = (byte & 0x80u) == 0;
    if (j >= 0 && start) emit(cur);
  }
}

// Sum of the numbers that end in the sixteen bytes.  Where a wave holds numbers
// of one and two bytes only, four bytes at a time: first bytes weigh 1, second
// bytes 128.  A byte 15 that continues belongs to the next thread; a byte 0
// that continues a number brings that number's first byte (h's last) with it.
__device__ __forceinline__ uint32_t sum_numbers(const Bytes16& b) {
  uint32_t s0 = 0, s1 = 0, prev = b.h, later_prev = (b.h << 8) & 0x80000000u;
  // deep: some number has a third byte (a byte and its predecessor both
  // continue a number), here or just past byte 15
  uint32_t deep = 0, first_later = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t later = __builtin_amdgcn_alignbit(b.w[q], prev, 24) & 0x80808080u;
    if (q == 0) first_later = later & 0x80u;
    deep |= later & __builtin_amdgcn_alignbit(later, later_prev, 24);
    prev = b.w[q];
    later_prev = later;
    const uint32_t m = (later << 1) - (later >> 7);  // 0xFF in later bytes
    const uint32_t v = b.w[q] & 0x7F7F7F7Fu;
    s0 = __builtin_amdgcn_sad_u8(v & ~m, 0u, s0);
    s1 = __builtin_amdgcn_sad_u8(v & m, 0u, s1);
  }
  deep |= later_prev & b.w[3] & 0x80000000u;
  uint32_t s = 0;
  if (__ballot(deep != 0u) == 0) {
    s = s0 + 128u * s1;
    if (b.w[3] >> 31) s -= (b.w[3] >> 24) & 0x7Fu;
    if (first_later) s += (b.h >> 24) & 0x7Fu;
  } else {
    walk_numbers(b, [&](uint32_t v) { s += v; });
  }
  return s;
}

__device__ __forceinline__ uint64_t stream_length(const uint64_t* n, uint64_t capacity) {
  const uint64_t x = *n;
  return x < capacity ? x : capacity;
}

// ---------------------------------------------------------------- COO pairs

// Sixteen pairs [q, q + 16) of a thread (q a multiple of 16; drow and dcol
// 16-byte aligned); pairs at or past n read as (0, 0) and are not used.
struct Pairs16 {
  uint32_t r[4];   // row fields, 4 per word
  uint32_t c[8];   // column fields, 2 per word
};

// This thread's sixteen pairs of the unit starting at q0 (none past q1; see
// "Prefetches" in stream_common.hpp).
__device__ __forceinline__ Pairs16 unit_pairs(const CooDecParams& p, uint64_t q0, uint64_t q1) {
  const uint64_t q = q0 + 16ull * threadIdx.x;
  const uint8_t* const zero = reinterpret_cast<const uint8_t*>(kStreamZero);
  const bool ok = q + 16 <= q1;
  const uint4 r = load16(ok ? p.drow + q : zero);
  const uint4 c0 = load16(ok ? reinterpret_cast<const uint8_t*>(p.dcol + q) : zero);
  const uint4 c1 = load16(ok ? reinterpret_cast<const uint8_t*>(p.dcol + q + 8) : zero);
  Pairs16 x;
  x.r[0] = r.x; x.r[1] = r.y; x.r[2] = r.z; x.r[3] = r.w;
  x.c[0] = c0.x; x.c[1] = c0.y; x.c[2] = c0.z; x.c[3] = c0.w;
  x.c[4] = c1.x; x.c[5] = c1.y; x.c[6] = c1.z; x.c[7] = c1.w;
  return x;
}

// The ragged sixteen of a unit [q0, q1) that ends the stream.
__device__ __forceinline__ void finish_pairs(Pairs16& x, const CooDecParams& p, uint64_t q0, uint64_t q1) {
  if (q1 - q0 == kDUnit) return;  // block-uniform
  const uint64_t q = q0 + 16ull * threadIdx.x;
  if (q >= q1 || q + 16 <= q1) return;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if (q + (uint64_t)j < q1) {
      x.r[j >> 2] |= (uint32_t)p.drow[q + j] << (8 * (j & 3));
      x.c[j >> 1] |= (uint32_t)p.dcol[q + j] << (16 * (j & 1));
    }
  }
}

__device__ __forceinline__ uint32_t pair_row(const Pairs16& x, int j) {
  return (x.r[j >> 2] >> (8 * (j & 3))) & 0xFFu;
}
__device__ __forceinline__ uint32_t pair_col(const Pairs16& x, int j) {
  return (x.c[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
}

// The map of one pair (see CooEl).
__device__ __forceinline__ CooEl pair_map(uint32_t dr, uint32_t dc) {
  if (dr == 255u && dc == 0u) return CooEl{0u, 1u, 255u, 0u, 1u};  // escape
  if (dr == 0u) return CooEl{0u, 1u, 0u, dc, 0u};
  return CooEl{0u, 0u, dr, dc - 1u, 0u};
}

// The absolute state at segment s's start: its first index as (row, column).
__device__ __forceinline__ CooEl segment_state(const CooDecParams& p, uint32_t s, uint32_t* C) {
  const uint32_t c = p.cols[s];
  *C = c > 0 ? c : 1u;
  const uint32_t f = p.first[s];
  const uint32_t row = f / *C;
  return CooEl{1u, 1u, row, f - row * *C, 0u};
}

struct CooLds {
  uint32_t seg[kDUnit / 32];     // segment starts among the unit's pairs
  uint32_t esc[kDUnit / 32];     // escape pairs
  uint64_t ref;                  // the position of the unit's first pair
  CooEl ws[kDWaves];
  SegCache cache;                // the segments whose pairs start in the tile
};

// The write pass's staging of a unit's entries.
struct CooStage {
  uint32_t val[padded(kDUnit)];  // flat index of each pair's entry (pair i at pad(i))
  uint32_t pos[padded(kDUnit)];  // low 32 bits of its position
};

// Writes segment s's first index at its first entry (if it has entries).
__device__ __forceinline__ void put_first(const CooDecParams& p, uint64_t nent, uint32_t s) {
  const uint64_t b = p.seg_begin[s];
  const uint64_t e = s + 1 < p.nseg ? p.seg_begin[s + 1] : nent;
  if (e > b && b < p.capacity) p.idx[b] = p.first[s];
}

// One unit of pairs [q0, q1) (q1 <= n; this thread's pairs x).  Returns carry
// combined with the unit's pairs.  WRITE: the entries are written, and the
// first index of every segment that starts in the unit (the last unit of the
// stream also those that start at its end).  Every thread of the block calls it.
template <bool WRITE>
__device__ CooEl coo_unit(const CooDecParams& p, const Pairs16& x, uint64_t q0, uint64_t q1, uint64_t n,
                          uint64_t nent, CooEl carry, bool last_unit, CooLds& L, CooStage* S) {
  const int tid = (int)threadIdx.x;
  const uint64_t q = q0 + 16ull * (uint64_t)tid;
  mark_unit(p.seg_pairs, L.cache, q0, q1, L.seg);
  uint32_t marks = run_marks(L.cache, L.seg);
  if (q == 0) marks |= 1u;  // the stream's first pair always starts a segment
  const uint32_t lo = L.cache.lo, hi = L.cache.lo + L.cache.n;
  const uint32_t m = q < q1 ? (uint32_t)(q1 - q < 16 ? q1 - q : 16) : 0u;  // this thread's pairs
  const uint32_t i0 = (uint32_t)tid * 16u;
  // this thread's map (absolute from its last segment start on)
  CooEl mine = CooEl::id();
  uint32_t C = 1;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if ((uint32_t)j < m) {
      if ((marks >> j) & 1u)
        mine = segment_state(p, segment_of(p.seg_pairs, L.cache, lo, hi, q + j), &C);
      mine = comb(mine, pair_map(pair_row(x, j), pair_col(x, j)));
    }
  }
  CooEl total;
  const CooEl before = block_scan_excl<kDT>(mine, carry, L.ws, &total);
  if (WRITE) {
    // Pair i's entry lands at seg_begin[s] + 1 + (pairs of s before it) -
    // (escapes of s before it).  Positions of one unit lie within
    // kDUnit + nseg < 2^31 of each other, so each is kept as its low 32 bits
    // beside the unit's first position.
    CooEl st = before;
    uint32_t s = 0;
    uint64_t sp = 0, sb = 0;
    C = 1;
    uint32_t escb = 0;
    if (m > 0) {
      s = segment_of(p.seg_pairs, L.cache, lo, hi, q);
      const uint32_t c = p.cols[s];
      C = c > 0 ? c : 1u;
      sp = p.seg_pairs[s];
      sb = p.seg_begin[s];
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if ((uint32_t)j < m) {
        const uint64_t qj = q + (uint64_t)j;
        if ((marks >> j) & 1u) {
          s = segment_of(p.seg_pairs, L.cache, lo, hi, qj);
          st = segment_state(p, s, &C);
          sp = p.seg_pairs[s];
          sb = p.seg_begin[s];
        }
        const uint32_t dr = pair_row(x, j), dc = pair_col(x, j);
        const uint64_t at = sb + 1 + (qj - sp) - st.e;
        st = comb(st, pair_map(dr, dc));
        if (dr == 255u && dc == 0u) escb |= 1u << j;
        S->val[pad(i0 + j)] = st.a * C + st.b;
        S->pos[pad(i0 + j)] = (uint32_t)at;
        if (qj == q0) L.ref = at;
      }
    }
    // two threads share a word: the even one holds its low half
    reinterpret_cast<uint16_t*>(L.esc)[tid] = (uint16_t)escb;
    __syncthreads();
    const uint64_t ref = L.ref;
    const uint32_t cnt = (uint32_t)(q1 - q0);
    for (uint32_t i = (uint32_t)tid; i < cnt; i += kDT) {
      if (bit_at(L.esc, i)) continue;  // an escape has no entry
      const uint64_t at = ref + (uint64_t)(int64_t)(int32_t)(S->pos[pad(i)] - (uint32_t)ref);
      if (at < p.capacity) p.idx[at] = S->val[pad(i)];
    }
    if (tid < 64) {
      for (uint32_t t = lo + (uint32_t)lane_id(); t < hi; t += 64) {
        const uint64_t v = start_of(p.seg_pairs, L.cache, t);
        if (v >= q0 && v < q1) put_first(p, nent, t);
      }
      if (last_unit) {
        const uint32_t from = lower_bound_wave(p.seg_pairs, p.nseg, n);
        for (uint32_t t = from + (uint32_t)lane_id(); t < p.nseg; t += 64) put_first(p, nent, t);
      }
    }
  }
  __syncthreads();  // the LDS arrays are rewritten by the next unit
  return total;
}

__device__ __forceinline__ void store_el(uint64_t* w, CooEl x) {
  w[0] = (uint64_t)x.a | ((uint64_t)x.b << 32);
  w[1] = (uint64_t)x.e | ((uint64_t)x.k << 32) | ((uint64_t)x.abs << 33);
}
__device__ __forceinline__ CooEl load_el(const uint64_t* w) {
  const uint64_t w0 = w[0], w1 = w[1];
  return CooEl{(uint32_t)(w1 >> 33) & 1u, (uint32_t)(w1 >> 32) & 1u, (uint32_t)w0,
               (uint32_t)(w0 >> 32), (uint32_t)w1};
}

}  // namespace

// ---------------------------------------------------------------- varint
//
// Table words, for tile b: word b its (entries | sum << 32); in the next two
// regions its first entry, and the running sum carried into it.

constexpr uint32_t kFirstWords = kMaxStreamTiles + 1;
constexpr uint32_t kCarryWords = 2 * (kMaxStreamTiles + 1);
static_assert(3 * (uint64_t)(kMaxStreamTiles + 1) <= kTableWords, "three words per tile");

__global__ __launch_bounds__(kDT) void varint_count_kernel(VarintDecParams p) {
  __shared__ uint32_t s_w[kDWaves];
  __shared__ uint32_t s_w2[kDWaves];
  const uint64_t n = stream_length(p.nbytes, p.in_capacity);
  const Geo g = stream_geometry(n);
  if (blockIdx.x >= g.ntiles) return;
  const uint64_t t0 = (uint64_t)blockIdx.x * g.tile;
  const uint64_t t1 = t0 + g.tile < n ? t0 + g.tile : n;
  uint32_t cnt = 0, sum = 0;
  for (uint64_t u0 = t0; u0 < t1; u0 += 4 * kDUnit) {
    // four units' loads in flight
    Bytes16 b[4];
#pragma unroll
    for (uint64_t q = 0; q < 4; ++q) b[q] = unit_bytes(p.in, u0 + q * kDUnit, t1);
#pragma unroll
    for (uint64_t q = 0; q < 4; ++q) {
      // (a unit past the tile would be walked byte by byte: 400M set's patch,
      // one-unit tiles, 20.8 us instead of 8)
      if (u0 + q * kDUnit >= t1) break;  // block-uniform
      finish_bytes(b[q], p.in, u0 + q * kDUnit, t1);
      cnt += terminators(b[q]);
      sum += sum_numbers(b[q]);
    }
  }
  // block sums of both
  const int lane = lane_id(), wid = (int)threadIdx.x >> 6;
  const uint32_t c = __builtin_amdgcn_readlane(wave_incl_scan(cnt), 63);
  const uint32_t s = __builtin_amdgcn_readlane(wave_incl_scan(sum), 63);
  if (lane == 0) {
    s_w[wid] = c;
    s_w2[wid] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t C = 0, S = 0;
    for (int w = 0; w < kDWaves; ++w) {
      C += s_w[w];
      S += s_w2[w];
    }
    stream_words(p.ws)[blockIdx.x] = (uint64_t)C | ((uint64_t)S << 32);
  }
}

// Entries and plain sum (modulo 2^32) before a tile.
struct Before {
  uint64_t cnt;
  uint32_t sum;
  __device__ static Before id() { return Before{0ull, 0u}; }
};
__device__ __forceinline__ Before comb(Before x, Before y) { return Before{x.cnt + y.cnt, x.sum + y.sum}; }
__device__ __forceinline__ Before shfl_up(Before x, int d) {
  return Before{(uint64_t)__shfl_up(x.cnt, d, 64), (uint32_t)__shfl_up((int)x.sum, d, 64)};
}

// Block s, s + grid, ...: segment s (and block 0 the entries before the first
// segment).  The tiles whose first entry lies past its start, up to its end,
// carry in the plain sum before them less the one before the segment: the
// block folds the tile words into LDS, searches the segment's tiles there, sums
// the numbers of the start's tile up to it, and writes those tiles' first
// entries and carries.  Every tile's first entry lies in exactly one segment's
// range.  What bounds it: the latency of the fold, then of each segment with
// such a tile (~2 us: its starts, its tile's bytes, the block sums).  Searching
// the tiles in registers, all of them for each segment, took as long again:
// decode of the 150M set's patch in 300 / 1,500 / 3,000 tensors 29.1 / 36.1 /
// 45.2 us, now 22.5 / 25.5 / 28.4.
__global__ __launch_bounds__(kDT) void varint_carry_kernel(VarintDecParams p) {
  __shared__ Before s_wb[kDWaves];
  __shared__ uint32_t s_w[kDWaves];
  __shared__ uint64_t s_cnt[padded(kMaxStreamTiles)];  // entries before each tile (tile i at pad(i))
  __shared__ uint32_t s_sum[padded(kMaxStreamTiles)];  // and their plain sum
  const uint64_t n = stream_length(p.nbytes, p.in_capacity);
  const Geo g = stream_geometry(n);
  uint64_t* words = stream_words(p.ws);
  const uint32_t per = (g.ntiles + kDT - 1) / kDT;  // tiles of a thread
  Before run = Before::id(), total;
  uint64_t x[kFoldPer];
#pragma unroll
  for (uint32_t q = 0; q < kFoldPer; ++q) {
    if (q >= per) break;  // block-uniform
    const uint32_t i = threadIdx.x * per + q;
    x[q] = i < g.ntiles ? words[i] : 0ull;
  }
#pragma unroll
  for (uint32_t q = 0; q < kFoldPer; ++q) {
    if (q >= per) break;
    run = comb(run, Before{(uint32_t)x[q], (uint32_t)(x[q] >> 32)});
  }
  Before at = block_scan_excl<kDT>(run, Before::id(), s_wb, &total);
#pragma unroll
  for (uint32_t q = 0; q < kFoldPer; ++q) {
    if (q >= per) break;
    const uint32_t i = threadIdx.x * per + q;
    if (i < g.ntiles) {
      s_cnt[pad(i)] = at.cnt;
      s_sum[pad(i)] = at.sum;
    }
    at = comb(at, Before{(uint32_t)x[q], (uint32_t)(x[q] >> 32)});
  }
  __syncthreads();
  // The first tile with more than e entries before it; every wave searches for itself.
  auto past = [&](uint64_t e) {
    return e == ~0ull ? g.ntiles
                      : lower_bound_wave([&](uint32_t i) { return s_cnt[pad(i)]; }, g.ntiles, e + 1);
  };
  auto segment = [&](uint64_t e, uint64_t next) {  // block-uniform
    const uint32_t i0 = e == 0 ? 0u : past(e), i1 = past(next);
    if (i0 >= i1) return;  // no tile's first entry lies in the segment
    uint32_t before = 0;  // the sum of all numbers before entry e
    if (e > 0) {
      const uint32_t tile = i0 - 1;  // holds entry e
      const uint32_t want = (uint32_t)(e - s_cnt[pad(tile)]);  // its entries before e
      const uint64_t t0 = (uint64_t)tile * g.tile;
      const uint64_t t1 = t0 + g.tile < n ? t0 + g.tile : n;
      uint32_t seen = 0, sum = 0;
      for (uint64_t u0 = t0; u0 < t1 && seen < want; u0 += kDUnit) {  // block-uniform
        Bytes16 b = unit_bytes(p.in, u0, t1);
        finish_bytes(b, p.in, u0, t1);
        uint32_t c;
        uint32_t k = seen + block_count_excl(terminators(b), s_w, &c);
        walk_numbers(b, [&](uint32_t v) {
          if (k < want) sum += v;
          ++k;
        });
        seen += c;
      }
      uint32_t all;
      (void)block_count_excl(sum, s_w, &all);
      before = s_sum[pad(tile)] + all;
    }
    for (uint32_t i = i0 + threadIdx.x; i < i1; i += kDT) {
      words[kFirstWords + i] = s_cnt[pad(i)];
      words[kCarryWords + i] = (uint64_t)(s_sum[pad(i)] - before);
    }
  };
  const uint32_t nseg = p.seg_begin ? p.nseg : 0u;
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) *p.count = total.cnt;
    const uint64_t first = nseg ? p.seg_begin[0] : ~0ull;
    if (first > 0) segment(0, first);
  }
  for (uint32_t s = blockIdx.x; s < nseg; s += gridDim.x) {
    const uint64_t e = p.seg_begin[s];
    const uint64_t next = s + 1 < nseg ? p.seg_begin[s + 1] : ~0ull;
    if (next <= e || (e > 0 && e >= total.cnt)) continue;  // empty, or past the last entry
    segment(e, next);
  }
}

__global__ __launch_bounds__(kDT) void varint_write_kernel(VarintDecParams p) {
  __shared__ uint32_t s_val[padded(kDUnit)];  // the unit's indices, in entry order (entry i at pad(i))
  __shared__ uint32_t s_bits[kDUnit / 32];
  __shared__ uint32_t s_w[kDWaves];
  __shared__ Sum64 s_wu[kDWaves];
  __shared__ SegSum s_ws[kDWaves];
  __shared__ SegCache s_seg;
  const int tid = (int)threadIdx.x;
  const uint64_t n = stream_length(p.nbytes, p.in_capacity);
  const Geo g = stream_geometry(n);
  if (blockIdx.x >= g.ntiles) return;
  uint64_t* words = stream_words(p.ws);
  const uint64_t t0 = (uint64_t)blockIdx.x * g.tile;
  const uint64_t t1 = t0 + g.tile < n ? t0 + g.tile : n;
  Bytes16 b = unit_bytes(p.in, t0, t1);
  const uint32_t ecnt = (uint32_t)words[blockIdx.x];
  const uint64_t e0 = words[kFirstWords + blockIdx.x];
  uint32_t carry = (uint32_t)words[kCarryWords + blockIdx.x];
  cache_tile_segments(p.seg_begin, p.nseg, e0, e0 + ecnt, s_seg);  // ends with a barrier: every
  if (tid == 0) {                                                  // thread has read the tile's words
    words[blockIdx.x] = 0;
    words[kFirstWords + blockIdx.x] = 0;
    words[kCarryWords + blockIdx.x] = 0;
  }
  uint64_t e = e0;
  for (uint64_t u0 = t0; u0 < t1; u0 += kDUnit) {
    const uint64_t u1 = u0 + kDUnit < t1 ? u0 + kDUnit : t1;
    Bytes16 cur = b;
    b = unit_bytes(p.in, u1, u1 + kDUnit < t1 ? u1 + kDUnit : t1);  // the next unit's, in flight
    finish_bytes(cur, p.in, u0, u1);
    // one walk: a number at the byte that ends it
    uint32_t v[16], ends = 0, sum = 0;
    {
      uint32_t cv = 0, sh = 0;
      bool begin = true;
#pragma unroll
      for (int j = -4; j < 16; ++j) {
        const uint32_t byte = j < 0 ? (cur.h >> (8 * (j + 4))) & 0xFFu : (cur.w[j >> 2] >> (8 * (j & 3))) & 0xFFu;
        const uint32_t v7 = byte & 0x7Fu;
        cv = begin ? v7 : cv | (sh < 32 ? v7 << sh : 0u);
        sh = begin ? 7 : sh + 7;
        begin = (byte & 0x80u) == 0;
        if (j >= 0) {
          v[j] = cv;
          ends |= begin ? 1u << j : 0u;
          sum += begin ? cv : 0u;
        }
      }
    }
    // this thread's rank among the unit's entries, and the sum before it
    const uint32_t mine = (uint32_t)__builtin_popcount(ends);
    uint32_t k, ucnt, acc, marks = 0;
    if (s_seg.n == 0) {
      // no segment starts in the tile: one scan of (sum, count); sums wrap out
      // of the top, and a unit's count never reaches bit 32
      Sum64 all;
      const uint64_t ex =
          block_scan_excl<kDT>(Sum64{((uint64_t)sum << 32) | mine}, Sum64::id(), s_wu, &all).v;
      k = (uint32_t)ex;
      ucnt = (uint32_t)all.v;
      acc = carry + (uint32_t)(ex >> 32);
      carry += (uint32_t)(all.v >> 32);
    } else {
      k = block_count_excl(mine, s_w, &ucnt);
      mark_unit(p.seg_begin, s_seg, e, e + ucnt, s_bits);
      SegSum own = SegSum::id();
      uint32_t r = k;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        if ((ends >> j) & 1u) {
          const bool at_start = bit_at(s_bits, r);
          marks |= at_start ? 1u << j : 0u;
          own = comb(own, SegSum{at_start ? 1u : 0u, v[j]});
          ++r;
        }
      }
      SegSum all;
      acc = block_scan_excl<kDT>(own, SegSum{0u, carry}, s_ws, &all).s;
      carry = all.s;
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if ((ends >> j) & 1u) {
        acc = (marks >> j) & 1u ? v[j] : acc + v[j];
        s_val[pad(k)] = acc;
        ++k;
      }
    }
    __syncthreads();
    for (uint32_t i = (uint32_t)tid; i < ucnt; i += kDT) {
      const uint64_t at = e + i;
      if (at < p.capacity) p.idx[at] = s_val[pad(i)];
    }
    e += ucnt;
    // no barrier here: the next unit writes s_val after its scan's barriers
  }
}

// ---------------------------------------------------------------- COO
//
// Table words 2b, 2b + 1: tile b's map, then its exclusive prefix.

__global__ __launch_bounds__(kDT) void coo_reduce_kernel(CooDecParams p) {
  __shared__ CooLds L;
  const uint64_t n = stream_length(p.npairs, p.pair_capacity);
  const uint64_t nent = *p.nent;
  const Geo g = stream_geometry(n);
  if (blockIdx.x >= g.ntiles) return;
  const uint64_t t0 = (uint64_t)blockIdx.x * g.tile;
  const uint64_t t1 = t0 + g.tile < n ? t0 + g.tile : n;
  Pairs16 x = unit_pairs(p, t0, t1);
  cache_tile_segments(p.seg_pairs, p.nseg, t0, t1, L.cache);
  CooEl run = CooEl::id();
  for (uint64_t u0 = t0; u0 < t1; u0 += kDUnit) {
    const uint64_t u1 = u0 + kDUnit < t1 ? u0 + kDUnit : t1;
    Pairs16 cur = x;
    x = unit_pairs(p, u1, u1 + kDUnit < t1 ? u1 + kDUnit : t1);  // the next unit's, in flight
    finish_pairs(cur, p, u0, u1);
    run = coo_unit<false>(p, cur, u0, u1, n, nent, run, false, L, nullptr);
  }
  if (threadIdx.x == 0) store_el(stream_words(p.ws) + 2ull * blockIdx.x, run);
}

// One block: the map before each tile.  (Folding the maps before its tile in
// every block of the write pass cost that pass 13 us on 1,128 tiles; this
// launch takes 5.)
__global__ __launch_bounds__(kST) void coo_scan_kernel(CooDecParams p) {
  __shared__ CooEl s_w[kST / 64];
  const uint64_t n = stream_length(p.npairs, p.pair_capacity);
  const Geo g = stream_geometry(n);
  uint64_t* w = stream_words(p.ws);
  auto ld = [&](uint32_t i) { return load_el(w + 2ull * i); };
  auto st = [&](uint32_t i, CooEl x) { store_el(w + 2ull * i, x); };
  single_block_scan<CooEl>(g.ntiles, ld, st, s_w);
}

__global__ __launch_bounds__(kDT) void coo_write_kernel(CooDecParams p) {
  __shared__ CooLds L;
  __shared__ CooStage S;
  const uint64_t n = stream_length(p.npairs, p.pair_capacity);
  const uint64_t nent = *p.nent;
  const Geo g = stream_geometry(n);
  if (blockIdx.x >= g.ntiles) return;
  const uint64_t t0 = (uint64_t)blockIdx.x * g.tile;
  const uint64_t t1 = t0 + g.tile < n ? t0 + g.tile : n;
  Pairs16 x = unit_pairs(p, t0, t1);
  uint64_t* const words = stream_words(p.ws) + 2ull * blockIdx.x;
  CooEl run = load_el(words);
  cache_tile_segments(p.seg_pairs, p.nseg, t0, t1, L.cache);  // ends with a barrier: every
  if (threadIdx.x == 0) {                                     // thread has read the tile's words
    words[0] = 0;
    words[1] = 0;
  }
  if (t0 >= t1) {  // the empty stream: only the segments' first indices
    run = coo_unit<true>(p, x, 0, 0, n, nent, run, true, L, &S);
  }
  for (uint64_t u0 = t0; u0 < t1; u0 += kDUnit) {
    const uint64_t u1 = u0 + kDUnit < t1 ? u0 + kDUnit : t1;
    Pairs16 cur = x;
    x = unit_pairs(p, u1, u1 + kDUnit < t1 ? u1 + kDUnit : t1);  // the next unit's, in flight
    finish_pairs(cur, p, u0, u1);
    run = coo_unit<true>(p, cur, u0, u1, n, nent, run, u1 == n, L, &S);
  }
}

// ---------------------------------------------------------------- launch

uint64_t stream_max_items() { return 1ull << 40; }

hipError_t launch_varint_decode(const VarintDecParams& p, hipStream_t stream) {
  const uint32_t grid = tile_grid(p.in_capacity);
  hipLaunchKernelGGL(varint_count_kernel, dim3(grid), dim3(kDT), 0, stream, p);
  if (hipError_t e = hipGetLastError()) return e;
  // as many blocks as are resident: each folds all tile words (3,000 segments of
  // the 150M set: 512 blocks 32.6 us, 768 28.4, 1,024 30.7)
  const uint32_t nseg = p.nseg < 1u ? 1u : p.nseg < 768u ? p.nseg : 768u;
  hipLaunchKernelGGL(varint_carry_kernel, dim3(nseg), dim3(kDT), 0, stream, p);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(varint_write_kernel, dim3(grid), dim3(kDT), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_coo_decode(const CooDecParams& p, hipStream_t stream) {
  const uint32_t grid = tile_grid(p.pair_capacity);
  hipLaunchKernelGGL(coo_reduce_kernel, dim3(grid), dim3(kDT), 0, stream, p);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(coo_scan_kernel, dim3(1), dim3(kST), 0, stream, p);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(coo_write_kernel, dim3(grid), dim3(kDT), 0, stream, p);
  return hipGetLastError();
}

}  // namespace pulse
