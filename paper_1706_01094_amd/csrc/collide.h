// Device helpers of the D1Q3 step kernels: the exact draw of a site's
// collision from the global tables, the literal sub-collision loop, the
// decision from a collision image in LDS, and accesses to a slot's arrays.
#pragma once
#include "device.h"
#include "rng.h"

namespace mclg {
namespace {

// Galilean-invariant acceptance of fiber (N, |J|) as a numerator over 2^32:
// floor(g num / den) with g = floor(2^32 N / sqrt(N^2 + 3 J^2)), both exact:
// each is estimated in double and corrected by integer tests that use only
// products (g is the largest integer with g^2 (N^2 + 3 J^2) <= 2^64 N^2).
__device__ uint64_t galilean_lambda(uint32_t num, uint32_t den, uint32_t N, uint32_t absJ) {
  using u128 = unsigned __int128;
  uint64_t g = 1ull << 32;
  if (absJ) {
    const uint64_t n2 = (uint64_t)N * N, d = n2 + 3ull * absJ * absJ;
    const u128 bound = (u128)n2 << 64;
    uint64_t s = (uint64_t)(4294967296.0 * (double)N / __dsqrt_rn((double)d));
    while (s && (u128)s * s * d > bound) --s;
    while ((u128)(s + 1) * (s + 1) * d <= bound) ++s;
    g = s;
  }
  const uint64_t gn = g * num;  // < 2^61
  uint64_t q = (uint64_t)((double)gn / (double)den);
  while (q && (u128)q * den > gn) --q;
  while ((u128)(q + 1) * den <= gn) ++q;
  return q;
}

// The paper's C sub-collisions one by one (Eq. (select), Eq. (omega)), with a
// block of random words per turn: a sub-collision takes two words or three,
// in order from the site's blocks, and the lanes keep the block of their next
// word and the one after it, so that a wave computes one block per
// sub-collision, for the lanes that go on to their next.  (With a block at
// every word that some lane has none for, which is almost every word, 1000
// lattices of 1000 sites, none of them in the image and half of them past
// n_max, took 234 us per step and take 58.)  False where a draw may be
// rejected, which takes more words; b is the new rest count otherwise.
__device__ __forceinline__ bool collide_turns(uint32_t a, uint32_t &b, uint32_t c,
                                              const StepParams &p, uint32_t x, uint32_t t,
                                              uint32_t rid) {
  const uint2 key = make_uint2((uint32_t)p.seed, (uint32_t)(p.seed >> 32));
  const uint32_t N = a + b + c;
  uint32_t at = 0, have = 0;  // the next word; w1 is block have - 1, w0 the one before
  uint4 w0 = make_uint4(0u, 0u, 0u, 0u), w1 = w0;
  bool sure = true;
  for (int32_t s = 0; s < p.C;) {
    if (have < (at >> 2) + 2u) {
      w0 = w1;
      w1 = philox10(make_uint4(x, t, rid, 2u | have << 2), key);
      if (++have < 2u) continue;
    }
    const bool two = (at & 2u) != 0u, one = (at & 1u) != 0u;
    const uint32_t t1 = two ? w0.w : w0.y, t2 = two ? w1.x : w0.z;
    const uint64_t m1 = (uint64_t)(one ? t1 : two ? w0.z : w0.x) * N;
    const uint64_t m2 = (uint64_t)(one ? t2 : t1) * (N - 1u);
    const uint32_t r1 = (uint32_t)(m1 >> 32);
    uint32_t r2 = (uint32_t)(m2 >> 32);
    r2 += (r2 >= r1);
    const int v1 = r1 < a ? -1 : (r1 < a + b ? 0 : 1);
    const int v2 = r2 < a ? -1 : (r2 < a + b ? 0 : 1);
    // 1: a {-1,+1} pair, -1: a {0,0} pair, 0: neither
    const int kind = v1 + v2 != 0 ? 0 : v1 != 0 ? 1 : -1;
    const uint32_t D = kind > 0 ? p.lam_q : 8u * p.lam_q;
    const uint64_t m3 = (uint64_t)(one ? two ? w1.y : w0.w : t2) * D;
    sure = sure && (uint32_t)m1 >= N && (uint32_t)m2 >= N - 1u && (!kind || (uint32_t)m3 >= D);
    at += kind ? 3u : 2u;
    const int d = (uint32_t)(m3 >> 32) < p.lam_p ? kind : 0;
    a -= d;
    b += 2 * d;
    c -= d;
    ++s;
  }
  return sure;
}

// The sub-collisions of a site with N > n_max.  Returns the new rest count.
// MANY: in turns (where such sites are rare, its code would only be in the
// way: 2^24 sites of density 50, 28.1 us per step without it and 28.5 with).
// GAL selects the Galilean-invariant acceptance (its own kernel
// instantiation, so that the plain kernel carries none of its code).
template <bool GAL, bool MANY>
__device__ __forceinline__ uint32_t collide_direct(uint32_t a, uint32_t b, uint32_t c,
                                                const StepParams &p, uint32_t x, uint32_t t,
                                                uint32_t rid) {
  if constexpr (!GAL && MANY) {
    uint32_t n = b;
    if (collide_turns(a, n, c, p, x, t, rid)) return n;
  }
  WordStream ws;
  ws.key = make_uint2((uint32_t)p.seed, (uint32_t)(p.seed >> 32));
  ws.x = x; ws.t = t; ws.rid = rid; ws.block = 0; ws.used = 4;
  const uint32_t N = a + b + c;
  if constexpr (GAL) {
    // lambda = lq / 2^32: a {-1,+1} pair is accepted when a word is below lq,
    // a {0,0} pair (lambda / 8) when a 35-bit uniform (w1 * 8 + w2 >> 29) is.
    const uint64_t lq = galilean_lambda(p.lam_p, p.lam_q, N, c > a ? c - a : a - c);
    for (int32_t s = 0; s < p.C; ++s) {
      const uint32_t r1 = ws.uniform(N);
      uint32_t r2 = ws.uniform(N - 1);
      r2 += (r2 >= r1);
      const int v1 = r1 < a ? -1 : (r1 < a + b ? 0 : 1);
      const int v2 = r2 < a ? -1 : (r2 < a + b ? 0 : 1);
      if (v1 + v2 == 0 && v1 != 0) {
        if ((uint64_t)ws.next() < lq) { a -= 1; c -= 1; b += 2; }
      } else if (v1 == 0 && v2 == 0) {
        const uint64_t w1 = ws.next();
        const uint32_t w2 = ws.next();
        if (((w1 << 3) | (w2 >> 29)) < lq) { b -= 2; a += 1; c += 1; }
      }
    }
    return b;
  }
  for (int32_t s = 0; s < p.C; ++s) {
    const uint32_t r1 = ws.uniform(N);
    uint32_t r2 = ws.uniform(N - 1);
    r2 += (r2 >= r1);
    const int v1 = r1 < a ? -1 : (r1 < a + b ? 0 : 1);
    const int v2 = r2 < a ? -1 : (r2 < a + b ? 0 : 1);
    if (v1 + v2 == 0 && v1 != 0) {
      if (ws.uniform(p.lam_q) < p.lam_p) { a -= 1; c -= 1; b += 2; }
    } else if (v1 == 0 && v2 == 0) {
      if (ws.uniform(8u * p.lam_q) < p.lam_p) { b -= 2; a += 1; c += 1; }
    }
  }
  return b;
}

// Number of entries <= r of an ascending array of n values: probe seven
// evenly spaced pivots at once, then count the one bucket left (all its
// loads at once) -- two rounds of independent loads for n <= 64.
__device__ __forceinline__ uint32_t count_le_wide(const uint32_t *__restrict__ t, uint32_t n,
                                                  uint32_t r) {
  uint32_t lo = 0;
  while (n > 8u) {
    const uint32_t s = (n + 7u) >> 3;  // bucket width; pivots t[lo + j s - 1]
    uint32_t c = 0;
#pragma unroll
    for (uint32_t j = 1; j < 8; ++j)
      c += (j * s <= n && t[lo + j * s - 1u] <= r) ? 1u : 0u;
    lo += c * s;
    n = min(s, n - c * s);
  }
  uint32_t c = 0;
#pragma unroll
  for (uint32_t j = 0; j < 8; ++j) c += (j < n && t[lo + j] <= r) ? 1u : 0u;
  return lo + c;
}

// Exact row of the global tables: the number of thresholds <= r.
// Rows of up to 16 thresholds (every row of C <= 7, most of larger C) are
// counted from four 16-byte loads issued together; the threshold pool is
// padded by 16 values so that these loads stay inside it.
__device__ __forceinline__ uint32_t count_le_16(const uint32_t *t, uint32_t n, uint32_t r) {
  uint4 q[4];
  for (int j = 0; j < 4; ++j) __builtin_memcpy(&q[j], t + 4 * j, 16);  // 4-byte aligned
  uint32_t c = 0;
#pragma unroll
  for (uint32_t j = 0; j < 16; ++j) {
    const uint4 &v = q[j >> 2];
    const uint32_t x = (j & 3) == 0 ? v.x : (j & 3) == 1 ? v.y : (j & 3) == 2 ? v.z : v.w;
    c += (j < n && x <= r) ? 1u : 0u;
  }
  return c;
}

// Two 16-bit lanes of a 32-bit register.
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

typedef short i16x2 __attribute__((ext_vector_type(2)));
// Index of the outcome of a draw r of row `row`.  The 64-byte row decides it
// unless some value equals the draw's top 15 bits (see LdsImage's records for
// the arithmetic); then, or without such rows, the exact thresholds do.  The
// row costs one line of memory and 11 to 15 words of arithmetic.
__device__ __forceinline__ uint32_t global_outcome(const TableDev &tab, uint32_t row, uint32_t r) {
  if (tab.row16) {
    const uint4 *q = tab.row16 + (size_t)row * (kRow16 / 8);
    const uint4 q0 = q[0], q1 = q[1], q2 = q[2];
    const uint32_t rh = r >> 17, rr = rh << 16 | rh;
    uint32_t w[16] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w,
                      q2.x, q2.y, q2.z, q2.w, 0u,   0u,   0u,   0u};
    const uint32_t kf = w[0] & 0x7fffu;
#pragma unroll
    for (int j = 0; j < 12; ++j) w[j] -= rr;
    i16x2 m = __builtin_bit_cast(i16x2, w[0]);
#pragma unroll
    for (int j = 1; j < 12; ++j) m = __builtin_elementwise_min(m, __builtin_bit_cast(i16x2, w[j]));
    // minus the number of values >= rh (byte 0: k_first, not counted)
    int g = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_perm(w[1], w[0], 0x0b0a0908u), 0x01010100, 0, false);
#pragma unroll
    for (int j = 2; j < 12; j += 2)
      g = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_perm(w[j + 1], w[j], 0x0b0a0908u), 0x01010101, g, false);
    uint32_t n = 23u;
    if (tab.row_words > 12u) {
      const uint4 q3 = q[3];
      w[12] = q3.x - rr; w[13] = q3.y - rr; w[14] = q3.z - rr; w[15] = q3.w - rr;
#pragma unroll
      for (int j = 12; j < 16; ++j) m = __builtin_elementwise_min(m, __builtin_bit_cast(i16x2, w[j]));
#pragma unroll
      for (int j = 12; j < 16; j += 2)
        g = __builtin_amdgcn_sdot4((int)__builtin_amdgcn_perm(w[j + 1], w[j], 0x0b0a0908u), 0x01010101, g, false);
      n = 31u;
    }
    if (m.x != (short)0x8000 && m.y != (short)0x8000) return kf + n + (uint32_t)g;
  }
  const uint2 d = tab.rowdesc[row];
  const uint32_t n = (d.y >> 16) - 1u;
  return (d.y & 0xffffu) +
         (n <= 16u ? count_le_16(tab.thr + d.x, n, r) : count_le_wide(tab.thr + d.x, n, r));
}

// The slot's collision image in LDS: a directory of (min(a,c), max(a,c))
// pairs whose last row and column stand for every pair out of range, then
// 16-byte records, nb + 1 per pair (the last one for every b out of range).
// A record decides the outcome exactly whenever the top 15 bits of r lie in
// its window and differ from all of its values.
// The image sits at LDS address 0 (the step kernels have no static LDS, so
// their dynamic LDS starts there) and is read by byte address.
struct LdsView {
  // dim_a, dim_c, 4 (dim_c + 1), b_lo and nb, each in both 16-bit halves
  uint32_t da2, dc2, w4, blo2, nb2;
  // records with a window start of their own (see LdsImage): the mask of
  // that field, the move with no value >= the draw, how many values there
  // are and their weights in the sum over the signs
  uint32_t ksm, base, span, weights;
};
typedef uint32_t lds_v4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const uint32_t lds_c32;
typedef __attribute__((address_space(3))) const lds_v4 lds_c4;
__device__ __forceinline__ uint32_t lds_u32(uint32_t addr) { return *(lds_c32 *)(size_t)addr; }
__device__ __forceinline__ uint4 lds_u4(uint32_t addr) {
  const lds_v4 v = *(lds_c4 *)(size_t)addr;
  return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ LdsView image_view(const ImageDesc &im) {
  LdsView lv;
  lv.da2 = im.dim_a * 0x10001u;
  lv.dc2 = im.dim_c * 0x10001u;
  lv.w4 = 4u * (im.dim_c + 1u) * 0x10001u;
  lv.blo2 = im.b_lo * 0x10001u;
  lv.nb2 = im.nb * 0x10001u;
  lv.ksm = im.fixed ? 0u : ~0u;
  lv.base = im.fixed ? (uint32_t)-4 : (uint32_t)-6;
  lv.span = im.fixed ? 7u : 6u;
  lv.weights = im.fixed ? ~0u : 0x00ffffffu;
  return lv;
}

// ---------------------------------------------------------------------------
// Wave-level helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t get16(const uint32_t (&w)[4], int e) {
  return (e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xffffu);
}
__device__ __forceinline__ void set16(uint32_t (&w)[4], int e, uint32_t v) {
  if (e & 1) w[e >> 1] = (w[e >> 1] & 0xffffu) | (v << 16);
  else w[e >> 1] = (w[e >> 1] & 0xffff0000u) | (v & 0xffffu);
}
// A slot's three arrays through one buffer resource: byte address =
// voff (per lane) + soff (wave-uniform, a scalar register).  Offsets stay
// 32-bit, and the per-lane part of a chunk's vector accesses is the same
// 16 * lane for every window.
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr int kRsrcWord3 = 0x00020000;  // raw buffer, 32-bit data format (gfx9)
// CP: the cache policy bits of the access (0, or kStreamingPolicy for
// states that do not fit the caches: non-temporal, the lines are not
// expected to be reused before they leave).
constexpr int kStreamingPolicy = 2;  // nt
template <int CP = 0>
__device__ __forceinline__ void bload4(Rsrc r, uint32_t voff, uint32_t soff, uint32_t (&v)[4]) {
  const auto q = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, CP);
  v[0] = q[0]; v[1] = q[1]; v[2] = q[2]; v[3] = q[3];
}
template <int CP = 0>
__device__ __forceinline__ void bstore4(Rsrc r, uint32_t voff, uint32_t soff,
                                        const uint32_t (&v)[4]) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 q = {v[0], v[1], v[2], v[3]};
  __builtin_amdgcn_raw_buffer_store_b128(q, r, (int)voff, (int)soff, CP);
}
__device__ __forceinline__ uint32_t bload2(Rsrc r, uint32_t voff, uint32_t soff) {
  return __builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, (int)soff, 0);
}
__device__ __forceinline__ void bstore2(Rsrc r, uint32_t voff, uint32_t soff, uint32_t v) {
  __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v, r, (int)voff, (int)soff, 0);
}
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Lanes with a == b, and with a > b (unsigned), as a mask in scalar registers.
__device__ __forceinline__ uint64_t lanes_eq(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_uicmp(a, b, 32);
}
__device__ __forceinline__ uint64_t lanes_gt(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_uicmp(a, b, 34);
}

// Exact outcome for a queued site: global row, or the literal loop.  It is
// only reached from the drain, outside the unrolled per-site code, so the
// hot loop stays small enough for the instruction cache.  `flag`: whether the
// site's errors count (a copy's extra sites hold meaningless counts near its
// ends).
template <bool GAL, bool MANY = true>
__device__ __forceinline__ uint32_t resolve_queued(const uint4 e, const StepParams &p,
                                                const TableDev &tab, uint32_t t, uint32_t rid,
                                                uint32_t *err, bool flag = true) {
  const uint32_t x = e.x, a = e.y & 0xffffu, b = e.y >> 16, c = e.z, r = e.w;
  const uint32_t N = a + b + c;
  if (N > 65535u) {  // a post-collision count might not fit: flagged, kept
    if (flag) atomicOr(err, kErrOverflow);
    return b;
  }
  if (p.C == 0 || N < 2u) return b;  // no collision
  if (N <= p.n_max) {
    // (n_0 keeps the parity of N - |J|, its own)
    return (b & 1u) + 2u * global_outcome(tab, collision_row(N, b, min(a, c)), r);
  }
  if (p.C < 0) {
    if (flag) atomicOr(err, kErrEqRange);
    return b;
  }
  return collide_direct<GAL, MANY>(a, b, c, p, x, t, rid);
}

// Decision of one site from the LDS image, in three phases so that the LDS
// reads of several sites are in flight together: (1) directory read, (2)
// record read, (3) decision.  There is no branch and no range test per site:
// the directory clamps min(a, c) to dim_a and max(a, c) to dim_c, whose row
// and column lead to never records, and b - b_lo (mod 2^16) is clamped to nb,
// every pair's never record.  A site outside the image (or of an absent
// pair, or with N > n_max) thus reads a never record, a site with N < 2 a
// record of move 0, and a site whose N does not fit 16 bits lies outside
// (the image holds N < 3072 only).
//
// A record holds the top 15 bits of consecutive thresholds of the site's
// fiber row, each with bit 15 set: T_0 .. T_7 of the window of seven moves
// around none (fixed records), or T_0 .. T_6 of a window of six moves and the
// move of its first state (the others).  With rh the top 15 bits of the draw,
// one 32-bit subtraction gives (0x8000 + T - rh) for two values at a time
// without a borrow between them: bit 15 says T >= rh, and 0x8000 that they
// are equal, when only the full threshold decides.  The number g of values
// >= rh is a sum over the sign bytes, and the move of Eq. (collcons) is
// d = (b - b') / 2 = g - 4 (b' has b's parity); g of none or of all means
// outside the window.
struct SiteLook {
  uint4 q;
};

// Phase 1 of sites 2J and 2J + 1 with 16-bit packed arithmetic.
template <int J>
__device__ __forceinline__ void site_dir_pair(uint32_t &row0, uint32_t &row1, u16x2 &bis,
                                              const uint32_t (&va)[4],
                                              const uint32_t (&vb)[4], const uint32_t (&vc)[4],
                                              const LdsView &lv) {
  const u16x2 a = __builtin_bit_cast(u16x2, va[J]), b = __builtin_bit_cast(u16x2, vb[J]),
              c = __builtin_bit_cast(u16x2, vc[J]);
  const u16x2 lo = __builtin_elementwise_min(__builtin_elementwise_min(a, c),
                                             __builtin_bit_cast(u16x2, lv.da2));
  // (4 times the clamped maximum stays below 2^16, so one shift does both)
  const uint32_t hi4 =
      __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_elementwise_max(a, c),
                                                             __builtin_bit_cast(u16x2, lv.dc2)))
      << 2;
  const uint32_t off = __builtin_bit_cast(
      uint32_t, lo * __builtin_bit_cast(u16x2, lv.w4) + __builtin_bit_cast(u16x2, hi4));
  bis = __builtin_elementwise_min(b - __builtin_bit_cast(u16x2, lv.blo2),
                                  __builtin_bit_cast(u16x2, lv.nb2));
  row0 = lds_u32(off & 0xffffu);
  row1 = lds_u32(off >> 16);
}

// Phase 2 of sites 2J and 2J + 1: record address = row + 16 x clamped b.
__device__ __forceinline__ void rec_pair(SiteLook &s0, SiteLook &s1, uint32_t row0, uint32_t row1,
                                         u16x2 bis) {
  const uint32_t b = __builtin_bit_cast(uint32_t, bis);
  uint32_t a0, a1;
  asm("v_mad_u32_u16 %0, %1, 16, %2" : "=v"(a0) : "v"(b), "v"(row0));
  asm("v_mad_u32_u16 %0, %1, 16, %2 op_sel:[1,0,0,0]" : "=v"(a1) : "v"(b), "v"(row1));
  s0.q = lds_u4(a0);
  s1.q = lds_u4(a1);
}

// Phase 3: d in the low 16 bits and the lanes whose record does not decide
// their draw (their d is meaningless).  FIXED: the image's records are fixed
// ones.
template <bool FIXED>
__device__ __forceinline__ uint32_t site_finish(const SiteLook &s, uint32_t r, const LdsView &lv,
                                                uint64_t &miss) {
  const uint32_t rh = r >> 17, rr = rh << 16 | rh;
  const uint32_t x = s.q.x - rr, y = s.q.y - rr, z = s.q.z - rr, w = s.q.w - rr;
  const i16x2 m = __builtin_elementwise_min(
      __builtin_elementwise_min(__builtin_bit_cast(i16x2, x), __builtin_bit_cast(i16x2, y)),
      __builtin_elementwise_min(__builtin_bit_cast(i16x2, z), __builtin_bit_cast(i16x2, w)));
  const uint32_t least = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(m, m.yx));
  // 0xff for every value >= rh
  const uint32_t p0 = __builtin_amdgcn_perm(z, y, 0x0b0a0908u);
  const uint32_t p1 = __builtin_amdgcn_perm(x, w, 0x0b0a0908u);
  if constexpr (FIXED) {
    const int d = __builtin_amdgcn_sdot4(
        (int)p1, -1, __builtin_amdgcn_sdot4((int)p0, -1, -4, false), false);
    miss = lanes_eq(least, 0x80008000u) | lanes_gt((uint32_t)(d + 3), 6u);
    return (uint32_t)d;
  }
  const int g = __builtin_amdgcn_sdot4((int)p1, (int)lv.weights,
                                       __builtin_amdgcn_sdot4((int)p0, -1, 0, false), false);
  miss = lanes_eq(least, 0x80008000u) | lanes_gt((uint32_t)(g - 1), lv.span - 1u);
  return (((uint32_t)((int32_t)s.q.x >> 16)) & lv.ksm) + lv.base + (uint32_t)g;
}

// Phase 3 of sites 2J and 2J + 1: d of both in one word (16-bit lanes).
template <bool FIXED>
__device__ __forceinline__ uint32_t finish_pair(const SiteLook &s0, const SiteLook &s1,
                                                uint32_t r0, uint32_t r1, const LdsView &lv,
                                                uint64_t &m0, uint64_t &m1) {
  const uint32_t d0 = site_finish<FIXED>(s0, r0, lv, m0), d1 = site_finish<FIXED>(s1, r1, lv, m1);
  return __builtin_amdgcn_perm(d1, d0, 0x05040100u);
}
// Sites 2J and 2J + 1 move by d: n_-1 and n_+1 gain d, n_0 loses 2d.
__device__ __forceinline__ void apply_pair(uint32_t &a, uint32_t &b, uint32_t &c, uint32_t dp) {
  const u16x2 d = __builtin_bit_cast(u16x2, dp);
  a = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) + d);
  c = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, c) + d);
  // (one multiply-add; the compiler would split it into a shift and a subtraction)
  asm("v_pk_mad_u16 %0, %1, %2, %0" : "+v"(b) : "v"(dp), "s"(0xfffefffeu));
}

}  // namespace
}  // namespace mclg
