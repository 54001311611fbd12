// hash.hip -- the weight-level integrity hash of App. J.4 on gfx950.
//
// The paper hashes the BF16 bit patterns of all parameters, concatenated in a
// fixed order, with SHA-256, so that a receiver can check the weights it
// rebuilt from a patch chain.  One SHA-256 over the whole stream is a single
// chain of compressions that no GPU can split, so the hash is a tree of
// SHA-256: the stream (each value's two bytes, low byte first) is cut into
// 16 KiB leaves and combined with the Merkle Tree Hash of RFC 6962, Sec. 2.1
// (leaf = SHA-256(0x00 || chunk), node = SHA-256(0x01 || left || right), the
// left subtree holding the largest power of two of leaves below the count).
//
// SHA-256 (FIPS 180-4) is 32-bit integer work: about 1,650 VALU operations per
// 64-byte block, ~26 per byte, so the kernel is bound by the vector ALU, not
// by HBM (it reads 2 bytes per parameter once).  One lane hashes one leaf;
// lanes of a wave hash neighbouring leaves, 16 KiB apart, and each lane reads
// its own 64-byte blocks with 16-byte loads, a block ahead.
//
// Kernels:
//   hash_setup_kernel  writes the tensor table and gathers the leaves that
//                      cross a tensor boundary into scratch slots;
//   hash_leaf_kernel   one lane per leaf: its digest;
//   hash_leaf_pair_kernel  the same for few leaves, two lanes' waves per leaf;
//   hash_tree_kernel   one block per 512 digests: the 9 tree levels above
//                      them, in LDS; the host repeats it until one remains.
#include "launch.hpp"

namespace pulse {
namespace {

// ---------------------------------------------------------------------------
// FIPS 180-4 constants from their definitions (5.3.3, 4.2.2): the first 32
// bits of the fractional parts of the square roots of the first 8 primes and
// of the cube roots of the first 64 primes, as integer Newton roots evaluated
// by the compiler.
constexpr uint64_t newton_root(unsigned __int128 v, int e) {
  unsigned __int128 y = (unsigned __int128)1 << 40;  // above every root taken here
  for (;;) {
    unsigned __int128 z = e == 2 ? (y + v / y) / 2 : (2 * y + v / (y * y)) / 3;
    if (z >= y) return (uint64_t)y;
    y = z;
  }
}

struct ShaConsts {
  uint32_t k[64];
  uint32_t h0[8];
};

constexpr ShaConsts make_sha_consts() {
  ShaConsts c{};
  int found = 0;
  for (uint64_t p = 2; found < 64; ++p) {
    bool prime = true;
    for (uint64_t d = 2; d * d <= p; ++d)
      if (p % d == 0) prime = false;
    if (!prime) continue;
    c.k[found] = (uint32_t)newton_root((unsigned __int128)p << 96, 3);
    if (found < 8) c.h0[found] = (uint32_t)newton_root((unsigned __int128)p << 64, 2);
    ++found;
  }
  return c;
}

constexpr ShaConsts kSha = make_sha_consts();
static_assert(kSha.h0[0] == 0x6a09e667u && kSha.k[0] == 0x428a2f98u && kSha.k[63] == 0xc67178f2u,
              "SHA-256 constants");

__device__ __forceinline__ uint32_t rotr(uint32_t x, int n) {
  return __builtin_amdgcn_alignbit(x, x, n);
}

// gfx950's three-input bitwise instruction: the 8-bit immediate is the truth
// table, indexed by (x << 2) | (y << 1) | z over the operand bits.
__device__ __forceinline__ uint32_t xor3(uint32_t x, uint32_t y, uint32_t z) {
  return __builtin_amdgcn_bitop3_b32(x, y, z, 0x96);
}
__device__ __forceinline__ uint32_t ch(uint32_t x, uint32_t y, uint32_t z) {  // x ? y : z
  return __builtin_amdgcn_bitop3_b32(x, y, z, 0xCA);
}
__device__ __forceinline__ uint32_t maj(uint32_t x, uint32_t y, uint32_t z) {  // majority
  return __builtin_amdgcn_bitop3_b32(x, y, z, 0xE8);
}

// One SHA-256 compression (FIPS 180-4, 6.2.2) of the 16 message words w into st.
__device__ __forceinline__ void sha256_block(uint32_t (&st)[8], uint32_t (&w)[16]) {
  uint32_t a = st[0], b = st[1], c = st[2], d = st[3];
  uint32_t e = st[4], f = st[5], g = st[6], h = st[7];
#pragma unroll
  for (int t = 0; t < 64; ++t) {
    uint32_t wt;
    if (t < 16) {
      wt = w[t];
    } else {
      const uint32_t x = w[(t - 15) & 15], y = w[(t - 2) & 15];
      const uint32_t s0 = xor3(rotr(x, 7), rotr(x, 18), x >> 3);
      const uint32_t s1 = xor3(rotr(y, 17), rotr(y, 19), y >> 10);
      wt = w[t & 15] + s0 + w[(t - 7) & 15] + s1;
      w[t & 15] = wt;
    }
    const uint32_t S1 = xor3(rotr(e, 6), rotr(e, 11), rotr(e, 25));
    const uint32_t t1 = h + S1 + ch(e, f, g) + kSha.k[t] + wt;
    const uint32_t S0 = xor3(rotr(a, 2), rotr(a, 13), rotr(a, 22));
    const uint32_t t2 = S0 + maj(a, b, c);
    h = g;
    g = f;
    f = e;
    e = d + t1;
    d = c;
    c = b;
    b = a;
    a = t1 + t2;
  }
  st[0] += a;
  st[1] += b;
  st[2] += c;
  st[3] += d;
  st[4] += e;
  st[5] += f;
  st[6] += g;
  st[7] += h;
}

// The 64 rounds alone, on wk[t] = message schedule word + round constant, which
// get(t / 4) hands out four at a time.
template <typename Get>
__device__ __forceinline__ void sha256_rounds(uint32_t (&st)[8], Get get) {
  uint32_t a = st[0], b = st[1], c = st[2], d = st[3];
  uint32_t e = st[4], f = st[5], g = st[6], h = st[7];
#pragma unroll
  for (int t4 = 0; t4 < 16; ++t4) {
    const uint4 q = get(t4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t wk = i == 0 ? q.x : i == 1 ? q.y : i == 2 ? q.z : q.w;
      const uint32_t S1 = xor3(rotr(e, 6), rotr(e, 11), rotr(e, 25));
      const uint32_t t1 = (h + wk) + S1 + ch(e, f, g);
      const uint32_t S0 = xor3(rotr(a, 2), rotr(a, 13), rotr(a, 22));
      const uint32_t t2 = S0 + maj(a, b, c);
      h = g;
      g = f;
      f = e;
      e = d + t1;
      d = c;
      c = b;
      b = a;
      a = t1 + t2;
    }
  }
  st[0] += a;
  st[1] += b;
  st[2] += c;
  st[3] += d;
  st[4] += e;
  st[5] += f;
  st[6] += g;
  st[7] += h;
}

__device__ __forceinline__ void sha256_init(uint32_t (&st)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) st[i] = kSha.h0[i];
}

typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef const __attribute__((address_space(1))) u32x4_a4* gvec;  // global memory
typedef const __attribute__((address_space(1))) uint32_t* gword;

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void hash_setup_kernel(HashSetupParams p) {
  if (blockIdx.x == 0 && threadIdx.x < p.nentries)
    p.table[p.first_entry + threadIdx.x] = p.entries[threadIdx.x];
  if (blockIdx.x >= p.njobs) return;
  const HashCopyJob j = p.jobs[blockIdx.x];
  uint16_t* dst = (uint16_t*)(p.scratch + j.dst);
  // eight loads in flight per thread (one at a time: 7.5 us for a full leaf)
  constexpr int kAt = 8;
  for (uint64_t i0 = threadIdx.x; i0 < j.count; i0 += kAt * blockDim.x) {
    uint16_t v[kAt];
#pragma unroll
    for (int q = 0; q < kAt; ++q) {
      const uint64_t i = i0 + (uint64_t)q * blockDim.x;
      v[q] = j.src[i < j.count ? i : 0];
    }
#pragma unroll
    for (int q = 0; q < kAt; ++q) {
      const uint64_t i = i0 + (uint64_t)q * blockDim.x;
      if (i < j.count) dst[i] = v[q];
    }
  }
}

// ---------------------------------------------------------------------------
// Leaf digests.  Message of leaf l: 0x00 followed by its len bytes.  Message
// word k (big-endian, FIPS 180-4 5.2.1) is the 4 bytes at message offset 4k,
// i.e. stream bytes 4k-1 .. 4k+2 of the leaf: the high byte of one 4-byte
// word of the source and three bytes of the next, put in order by one
// v_perm_b32.  A leaf whose source starts 2 bytes into a word (after a tensor
// of odd length) takes the other byte selector.
struct LeafSource {
  // base[0 .. dmax] hold the leaf's bytes, starting sh bytes into base[0];
  // message word k pairs base[k - 1 + o] with base[k + o] by selector sel
  const uint32_t* base;
  uint32_t sel, prev, o, dmax;
  uint32_t len;  // bytes
};

__device__ __forceinline__ LeafSource leaf_source(const HashLeafParams& p, uint64_t l) {
  const uint64_t x = l * kHashLeafElems;
  const uint64_t le = p.total - x < kHashLeafElems ? p.total - x : kHashLeafElems;
  LeafSource s;
  s.len = (uint32_t)(2 * le);
  uint32_t lo = 0, hi = p.ntensors;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (p.table[mid].off <= x) lo = mid;
    else hi = mid;
  }
  const HashEntry t = p.table[lo];
  const uint64_t end = p.table[lo + 1].off;
  if (hash_leaf_in_place(x, le, t.off, end)) {
    const uintptr_t A = (uintptr_t)(t.ptr + (x - t.off));
    const uint32_t sh = (uint32_t)(A & 3);  // 0 or 2
    s.base = (const uint32_t*)(A - sh);
    s.o = sh >> 1;
    s.prev = sh ? (s.base[0] & 0xFFFF0000u) : 0u;  // the bytes before the leaf read as the prefix 0
    s.sel = sh ? 0x05060700u : 0x07000102u;
    s.dmax = (sh + s.len + 3) / 4 - 1;
  } else {
    s.base = (const uint32_t*)(p.scratch + (uint64_t)lo * kHashLeafBytes);
    s.o = 0;
    s.prev = 0u;
    s.sel = 0x07000102u;
    s.dmax = (s.len + 3) / 4 - 1;
  }
  return s;
}

// Blocks of a leaf's message of len + 1 bytes (the prefix): those made of
// message bytes only, and all of them with the padding.
__device__ __forceinline__ uint32_t full_blocks(uint32_t len) { return (len + 1) / 64; }
__device__ __forceinline__ uint32_t all_blocks(uint32_t len) { return (len + 1 + 1 + 8 + 63) / 64; }

// Block b of the message's end: its tail, the byte 0x80, zeros and the bit
// length (FIPS 180-4 5.1.1).  Reads are clamped to base[dmax]; the bytes past
// the message that such a read brings in are masked off.
__device__ __forceinline__ void tail_block(const LeafSource& s, uint32_t b, uint32_t& prev, uint32_t (&w)[16]) {
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint32_t k = 16 * b + j;
    const uint32_t cur = ((gword)s.base)[k + s.o < s.dmax ? k + s.o : s.dmax];
    uint32_t word = __builtin_amdgcn_perm(prev, cur, s.sel);
    prev = cur;
    const int nb = (int)(s.len + 1) - (int)(4 * k);  // message bytes left at this word
    word &= nb >= 4 ? 0xFFFFFFFFu : nb <= 0 ? 0u : ~(0xFFFFFFFFu >> (8 * nb));
    if (nb >= 0 && nb < 4) word |= 0x80u << (24 - 8 * nb);
    w[j] = word;
  }
  if (b == all_blocks(s.len) - 1) {
    w[14] = 0;
    w[15] = 8 * (s.len + 1);
  }
}

__device__ __forceinline__ void store_digest(uint8_t* digests, uint64_t l, const uint32_t (&st)[8]) {
  uint32_t* out = (uint32_t*)(digests + 32 * l);
  u32x4_a4 o0 = {__builtin_bswap32(st[0]), __builtin_bswap32(st[1]), __builtin_bswap32(st[2]),
                 __builtin_bswap32(st[3])};
  u32x4_a4 o1 = {__builtin_bswap32(st[4]), __builtin_bswap32(st[5]), __builtin_bswap32(st[6]),
                 __builtin_bswap32(st[7])};
  *(u32x4_a4*)out = o0;
  *(u32x4_a4*)(out + 4) = o1;
}

__global__ __launch_bounds__(256) void hash_leaf_kernel(HashLeafParams p) {
  const uint64_t l = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= p.nleaves) return;
  const LeafSource src = leaf_source(p, l);
  const uint32_t nfull = full_blocks(src.len);
  uint32_t prev = src.prev;
  uint32_t st[8];
  sha256_init(st);
  uint32_t d[16];
  auto load = [&](const uint32_t* at) {
    const gvec q = (gvec)at;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4_a4 v = __builtin_nontemporal_load(q + i);
      d[4 * i] = v.x;
      d[4 * i + 1] = v.y;
      d[4 * i + 2] = v.z;
      d[4 * i + 3] = v.w;
    }
  };
  // The next block's loads are in flight during each compression: with few waves
  // per SIMD nothing else hides them (0.5B set 982 -> 895 us, 7B set 10.87 ->
  // 10.76 ms).
  if (nfull > 0) load(src.base + src.o);
  for (uint32_t b = 0; b < nfull; ++b) {
    uint32_t w[16];
    w[0] = __builtin_amdgcn_perm(prev, d[0], src.sel);
#pragma unroll
    for (int j = 1; j < 16; ++j) w[j] = __builtin_amdgcn_perm(d[j - 1], d[j], src.sel);
    prev = d[15];
    load(src.base + 16 * (b + 1 < nfull ? b + 1 : b) + src.o);
    sha256_block(st, w);
  }
  const uint32_t nblocks = all_blocks(src.len);
  for (uint32_t b = nfull; b < nblocks; ++b) {
    uint32_t w[16];
    tail_block(src, b, prev, w);
    sha256_block(st, w);
  }
  store_digest(p.digests, l, st);
}

// Few leaves: two waves per 64 leaves.  A leaf is one chain of 257 blocks, and a
// SIMD with one wave of such chains issues an instruction every five cycles (at
// best every four), however little there is to hash.  One wave forms the
// message schedules, a block ahead, and leaves them in LDS with the round
// constants added; the other has only the rounds to do.  Whole call, one wave
// per 64 leaves / two: 1M values 691 / 531 us, 200M 855 / 667; where a CU gets
// more than one such block (four waves, 128 leaves) the pairs lose: 300M
// 881 / 940.
constexpr uint64_t kPairLeaves = 128ull * 256;  // one block on each of the 256 CUs
__device__ __align__(16) const uint32_t kHashZero[16] = {0};

__global__ __launch_bounds__(256) void hash_leaf_pair_kernel(HashLeafParams p) {
  __shared__ uint4 s_wk[2][2][16][64];  // [buffer][pair][schedule words 4 i .. 4 i + 3][leaf]
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  // two pairs per block, a wave on each SIMD
  const uint32_t pair = wave & 1u;
  const bool schedules = wave >= 2;
  const uint64_t b0 = (uint64_t)blockIdx.x * 128, l0 = b0 + pair * 64;
  const uint64_t l = l0 + lane < p.nleaves ? l0 + lane : p.nleaves - 1;  // (the last one again)
  // the block's first leaf is its longest: all waves walk that many blocks
  const uint64_t x0 = b0 * kHashLeafElems;
  const uint32_t nb = all_blocks((uint32_t)(2 * (p.total - x0 < kHashLeafElems ? p.total - x0 : kHashLeafElems)));
  if (schedules) {
    const LeafSource src = leaf_source(p, l);
    const uint32_t nfull = full_blocks(src.len);
    uint32_t prev = src.prev;
    uint32_t d[16];
    auto load = [&](uint32_t b) {  // unconditional, so that it stays in flight
      const gvec q = (gvec)(b < nfull ? src.base + 16 * b + src.o : kHashZero);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const u32x4_a4 v = q[i];
        d[4 * i] = v.x;
        d[4 * i + 1] = v.y;
        d[4 * i + 2] = v.z;
        d[4 * i + 3] = v.w;
      }
    };
    load(0);
    for (uint32_t b = 0; b < nb; ++b) {
      uint32_t w[16];
      if (b < nfull) {
        w[0] = __builtin_amdgcn_perm(prev, d[0], src.sel);
#pragma unroll
        for (int j = 1; j < 16; ++j) w[j] = __builtin_amdgcn_perm(d[j - 1], d[j], src.sel);
        prev = d[15];
      } else {
        tail_block(src, b, prev, w);
      }
      load(b + 1);
      uint4(*const to)[64] = s_wk[b & 1][pair];
#pragma unroll
      for (int t4 = 0; t4 < 16; ++t4) {
        uint32_t wk[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = 4 * t4 + i;
          if (t >= 16) {
            const uint32_t x = w[(t - 15) & 15], y = w[(t - 2) & 15];
            const uint32_t s0 = xor3(rotr(x, 7), rotr(x, 18), x >> 3);
            const uint32_t s1 = xor3(rotr(y, 17), rotr(y, 19), y >> 10);
            w[t & 15] = w[t & 15] + s0 + w[(t - 7) & 15] + s1;
          }
          wk[i] = w[t & 15] + kSha.k[t];
        }
        to[t4][lane] = make_uint4(wk[0], wk[1], wk[2], wk[3]);
      }
      __syncthreads();  // block b is in buffer b & 1; the rounds of block b - 1 are done
    }
    return;
  }
  const uint32_t nblocks = l0 + lane < p.nleaves ? all_blocks((uint32_t)(2 * (p.total - l * kHashLeafElems < kHashLeafElems
                                                                                  ? p.total - l * kHashLeafElems
                                                                                  : kHashLeafElems)))
                                                 : 0u;
  uint32_t st[8];
  sha256_init(st);
  for (uint32_t b = 0; b < nb; ++b) {
    __syncthreads();
    const uint4(*const from)[64] = s_wk[b & 1][pair];
    if (b < nblocks) sha256_rounds(st, [&](int t4) { return from[t4][lane]; });
  }
  if (l0 + lane < p.nleaves) store_digest(p.digests, l, st);
}

// ---------------------------------------------------------------------------
// Interior node: SHA-256 of the 65 bytes 0x01 || L || R (two blocks).  L and R
// are digests as eight big-endian words, so the message words are L and R
// shifted right by one byte across word boundaries.
//
// The second block holds R's last byte and the padding: its message schedule
// is one of 256, kept with the round constants added.  A tree level is one
// chain of two compressions in a wave with a SIMD of its own (an instruction
// every five cycles), so the schedule's instructions are time; the row's loads
// are issued before the first block's rounds, which cover them.  Seven levels
// (118 nodes to 1): 36 -> 32 us; the 0.5B set's nine and seven: 102 -> 94 us.
struct TailRows {
  uint32_t wk[64][64];
};

// Rows of last bytes 64 part .. 64 part + 63.
constexpr TailRows make_tail_rows(uint32_t part) {
  TailRows t{};
  for (uint32_t r = 0; r < 64; ++r) {
    uint32_t w[64] = {};
    w[0] = ((64 * part + r) << 24) | 0x00800000u;
    w[15] = 65 * 8;
    for (int i = 0; i < 64; ++i) {
      if (i >= 16) {
        const uint32_t x = w[i - 15], y = w[i - 2];
        w[i] = w[i - 16] + ((x >> 7 | x << 25) ^ (x >> 18 | x << 14) ^ (x >> 3)) + w[i - 7] +
               ((y >> 17 | y << 15) ^ (y >> 19 | y << 13) ^ (y >> 10));
      }
      t.wk[r][i] = w[i] + kSha.k[i];
    }
  }
  return t;
}

__device__ __align__(16) constexpr TailRows kTail[4] = {make_tail_rows(0), make_tail_rows(1),
                                                        make_tail_rows(2), make_tail_rows(3)};

__device__ __forceinline__ void node_hash(const uint32_t (&L)[8], const uint32_t (&R)[8],
                                          uint32_t (&st)[8]) {
  const uint4* const row = reinterpret_cast<const uint4*>(&kTail[0].wk[0][0] + 64 * (R[7] & 0xFFu));
  uint4 q[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) q[i] = row[i];
  __builtin_amdgcn_sched_barrier(0);
  sha256_init(st);
  uint32_t w[16];
  w[0] = 0x01000000u | (L[0] >> 8);
#pragma unroll
  for (int i = 1; i < 8; ++i) w[i] = __builtin_amdgcn_alignbit(L[i - 1], L[i], 8);
  w[8] = __builtin_amdgcn_alignbit(L[7], R[0], 8);
#pragma unroll
  for (int i = 9; i < 16; ++i) w[i] = __builtin_amdgcn_alignbit(R[i - 9], R[i - 8], 8);
  sha256_block(st, w);
  sha256_rounds(st, [&](int t4) { return q[t4]; });
}

__global__ __launch_bounds__(256) void hash_tree_kernel(const uint8_t* in, uint64_t n_in,
                                                        uint8_t* out) {
  __shared__ uint32_t s[2][kHashTreeFan][8];
  const uint32_t tid = threadIdx.x;
  if (n_in == 0) {  // no leaves: the hash of the empty message
    if (blockIdx.x == 0 && tid == 0) {
      uint32_t st[8], w[16];
      sha256_init(st);
      w[0] = 0x80000000u;
#pragma unroll
      for (int i = 1; i < 16; ++i) w[i] = 0;
      sha256_block(st, w);
#pragma unroll
      for (int i = 0; i < 8; ++i) ((uint32_t*)out)[i] = __builtin_bswap32(st[i]);
    }
    return;
  }
  const uint64_t base = (uint64_t)blockIdx.x * kHashTreeFan;
  uint32_t m = (uint32_t)(n_in - base < kHashTreeFan ? n_in - base : kHashTreeFan);
  const uint32_t* src = (const uint32_t*)(in + 32 * base);
  for (uint32_t i = tid; i < m * 8; i += blockDim.x)
    s[0][i >> 3][i & 7] = __builtin_bswap32(src[i]);
  __syncthreads();
  int cur = 0;
  // Pair neighbours level by level and carry an unpaired last node up as it
  // is: the same tree as RFC 6962's split at the largest power of two.
  while (m > 1) {
    const uint32_t half = (m + 1) / 2;
    if (tid < half) {
      uint32_t st[8];
      if (2 * tid + 1 < m) {
        uint32_t L[8], R[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          L[i] = s[cur][2 * tid][i];
          R[i] = s[cur][2 * tid + 1][i];
        }
        node_hash(L, R, st);
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) st[i] = s[cur][2 * tid][i];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) s[cur ^ 1][tid][i] = st[i];
    }
    __syncthreads();
    cur ^= 1;
    m = half;
  }
  if (tid < 8) ((uint32_t*)(out + 32 * (uint64_t)blockIdx.x))[tid] = __builtin_bswap32(s[cur][0][tid]);
}

}  // namespace

hipError_t launch_hash_setup(const HashSetupParams& p, hipStream_t stream) {
  const uint32_t grid = p.njobs > 0 ? p.njobs : 1;
  hipLaunchKernelGGL(hash_setup_kernel, dim3(grid), dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_hash_leaves(const HashLeafParams& p, hipStream_t stream) {
  if (p.nleaves == 0) return hipSuccess;
  if (p.nleaves <= kPairLeaves) {
    hipLaunchKernelGGL(hash_leaf_pair_kernel, dim3((uint32_t)((p.nleaves + 127) / 128)), dim3(256), 0, stream, p);
    return hipGetLastError();
  }
  const uint64_t grid = (p.nleaves + 255) / 256;
  hipLaunchKernelGGL(hash_leaf_kernel, dim3((uint32_t)grid), dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_hash_tree(const uint8_t* in, uint64_t n_in, uint8_t* out, hipStream_t stream) {
  const uint64_t grid = n_in == 0 ? 1 : (n_in + kHashTreeFan - 1) / kHashTreeFan;
  hipLaunchKernelGGL(hash_tree_kernel, dim3((uint32_t)grid), dim3(256), 0, stream, in, n_in, out);
  return hipGetLastError();
}

}  // namespace pulse
