// HIP kernels of the D2Q9 path of the MCLG library (Sec. "A D2Q9
// implementation"): one thread per site runs the literal loop of C
// sub-collisions with the rule table in LDS, in place in the shifted 2D
// layout; Poisson start, counts start, exact moments and histograms.  The
// rules and the layout are stated in mclg.h.
#include "d2q9.h"
#include "device.h"
#include "rng.h"

#include <algorithm>

namespace mclg {
namespace {

// ---- D2Q9 --------------------------------------------------------------
// Step9::rules holds the rules in the form device_rules9 builds (d2q9.h).
__constant__ int32_t kV9x[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__constant__ int32_t kV9y[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

// Physical element of velocity i of logical site s = y Lx + x at shift
// (tx, ty): ((x - vx tx) mod Lx, (y - vy ty) mod Ly), element y' Lx + x'.
// The row offsets y' Lx are (y Lx -/+ ty Lx) mod S, with y Lx = s - x.
struct Site9 {
  uint32_t e[9];
  __device__ Site9(uint32_t s, uint32_t x, uint32_t tx, uint32_t ty, uint32_t Lx, uint32_t S) {
    const uint32_t xs[3] = {x + tx >= Lx ? x + tx - Lx : x + tx, x, x >= tx ? x - tx : x + Lx - tx};
    const uint32_t yL = s - x, tyL = ty * Lx;
    const uint32_t rows[3] = {yL + tyL >= S ? yL + tyL - S : yL + tyL, yL,
                              yL >= tyL ? yL - tyL : yL + S - tyL};
#pragma unroll
    for (int i = 0; i < 9; ++i) e[i] = rows[kV9y[i] + 1] + xs[kV9x[i] + 1];
  }
};

// Element e (below 2^28) of velocity i: a uniform base and a 32-bit offset.
__device__ __forceinline__ uint16_t *at9(uint16_t *state, const Rep9 &rp, int i, uint32_t e) {
  char *const base = reinterpret_cast<char *>(state + rp.off + (uint64_t)i * rp.stride);
  return reinterpret_cast<uint16_t *>(base + 2u * e);
}

// Packed pairs of 16-bit partial sums (element 0 = low half).
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u16x2 as_u16x2(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ __forceinline__ uint32_t as_u32(u16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// #{j < 8 : K_j <= r} for the partial sums K held as four 16-bit pairs and
// r < 65535: max(0, r + 1 - K_j) is at least 1 exactly when K_j <= r.  `one`
// holds 1 in both halves; passed in a register it keeps the saturated
// difference and the minimum as two packed instructions per pair.
__device__ __forceinline__ uint32_t count_partial_le(const u16x2 (&K)[4], uint32_t r, u16x2 one) {
  const u16x2 R = as_u16x2((r + 1u) * 0x10001u);
  u16x2 acc = __builtin_elementwise_min(__builtin_elementwise_sub_sat(R, K[0]), one);
#pragma unroll
  for (int m = 1; m < 4; ++m) acc += __builtin_elementwise_min(__builtin_elementwise_sub_sat(R, K[m]), one);
  return (uint32_t)acc.x + (uint32_t)acc.y;
}

// Philox blocks (s, t, replica, 2 | sub << 2) of one site, words 0 to 2.  What
// does not depend on sub is computed once per site: the products of the first
// round, one of the second and one of the third (16 wide products of 20, and
// five exclusive ors of two words in place of three).
struct SiteBlocks {
  uint2 key;
  uint32_t z1, x3, x4;  // of the site
  uint32_t s2, s3;      // uniform
  static constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u, kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;
  __device__ SiteBlocks(uint2 k, uint32_t s, uint32_t t, uint32_t rid) : key(k) {
    const uint64_t p0 = (uint64_t)kM0 * s, p1 = (uint64_t)kM1 * rid;
    z1 = (uint32_t)(p0 >> 32) ^ k.y;
    const uint64_t q0 = (uint64_t)kM0 * ((uint32_t)(p1 >> 32) ^ t ^ k.x);
    s2 = (uint32_t)p1 ^ (k.x + kW0);
    const uint32_t z2 = (uint32_t)(q0 >> 32) ^ (uint32_t)p0 ^ (k.y + kW1);
    const uint64_t r1 = (uint64_t)kM1 * z2;
    x3 = (uint32_t)(r1 >> 32) ^ (k.x + 2u * kW0);
    s3 = (uint32_t)q0 ^ (k.y + 2u * kW1);
    x4 = (uint32_t)r1 ^ (k.x + 3u * kW0);
    asm volatile("" : "+v"(z1), "+v"(x3), "+v"(x4));
  }
  __device__ uint4 operator()(uint32_t sub) const {
    uint2 k = make_uint2(key.x + 3u * kW0, key.y + 3u * kW1);
    uint64_t p0, p1 = (uint64_t)kM1 * (z1 ^ (2u | sub << 2));
    p0 = (uint64_t)kM0 * ((uint32_t)(p1 >> 32) ^ s2);
    const uint32_t c3x = x3 ^ (uint32_t)p1, c3z = (uint32_t)(p0 >> 32) ^ s3, c3w = (uint32_t)p0;
    p0 = (uint64_t)kM0 * c3x;
    p1 = (uint64_t)kM1 * c3z;
    uint4 c = make_uint4((uint32_t)(p1 >> 32) ^ x4, (uint32_t)p1, xor3((uint32_t)(p0 >> 32), c3w, k.y), (uint32_t)p0);
#pragma unroll
    for (int i = 4; i < 10; ++i) {
      k.x += kW0;
      k.y += kW1;
      // recomputed at every use (scalar adds) rather than held in registers
      asm volatile("" : "+s"(k.x), "+s"(k.y));
      p0 = (uint64_t)kM0 * c.x;
      p1 = (uint64_t)kM1 * c.z;
      c = make_uint4(xor3((uint32_t)(p1 >> 32), c.y, k.x), (uint32_t)p1, xor3((uint32_t)(p0 >> 32), c.w, k.y), (uint32_t)p0);
    }
    return c;
  }
};

// The draws of a sub-collision: r[0] in [0, N), r[1] in [0, N - 1), r[2] in
// [0, D) from the block's words (multiply and reject, Lemire 2019).  Words
// that replace rejected ones come in order from the blocks
// (s, t, replica, 2 | (C + j) << 2); `used` of them are gone.  Each is
// computed where it is needed, so that a site carries one register for them.
template <bool QUOT>
__device__ __forceinline__ void draws(uint32_t (&r)[3], uint4 w, uint32_t N, const Step9 &a,
                                      uint32_t s, uint32_t rid, uint32_t &used) {
  const uint2 key = make_uint2((uint32_t)a.seed, (uint32_t)(a.seed >> 32));
  uint64_t m[3] = {(uint64_t)w.x * N, (uint64_t)w.y * (N - 1u), (uint64_t)w.z * a.D};
#pragma unroll
  for (int i = 0; i < 3; ++i) r[i] = (uint32_t)(m[i] >> 32);
  // floor(floor(z D / 2^32) / (D / Dq)) = floor(z Dq / 2^32)
  if (QUOT) {
    const uint64_t mq = (uint64_t)w.z * a.Dq;
    r[2] = (uint32_t)(mq >> 32);
    // (unused halves kept: one wide product costs a quarter of a high or a
    // low one)
    asm volatile("" : : "v"((uint32_t)mq), "v"((uint32_t)(m[2] >> 32)));
  }
  asm volatile("" : : "v"(w.w));
  // a draw is rejected with probability below 2^-16 for N and D up to 2^15:
  // one test of the smallest low product against the largest bound
  if (__builtin_expect(min(min((uint32_t)m[0], (uint32_t)m[1]), (uint32_t)m[2]) < max(N, a.D), 0)) {
#pragma unroll 1
    for (int i = 0; i < 3; ++i) {
      const uint32_t n = i == 0 ? N : i == 1 ? N - 1u : a.D;
      uint64_t p = (uint64_t)(i == 0 ? w.x : i == 1 ? w.y : w.z) * n;
      if ((uint32_t)p < n) {
        const uint32_t floor_ = (0u - n) % n;
        while ((uint32_t)p < floor_) {
          const uint4 v = philox10(
              make_uint4(s, (uint32_t)a.t, rid, 2u | (((uint32_t)a.C + (used >> 2)) << 2)), key);
          p = (uint64_t)word_of(v, used & 3u) * n;
          ++used;
        }
      }
      const uint32_t h = (uint32_t)(p >> 32);
      r[0] = i == 0 ? h : r[0];
      r[1] = i == 1 ? h : r[1];
      r[2] = i == 2 ? (QUOT ? h / (a.D / a.Dq) : h) : r[2];
    }
  }
  asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]));  // compared as 32-bit values
  r[1] += (r[1] >= r[0]);
}

// The sub-collision loop of one site with N < 2^7 (W = 2: bytes) or 2^15
// (W = 4: halves) particles, Dq <= 2^15.  Bound by the vector instructions:
// 69 of them (bytes; 100 with packed 16-bit sums for all), 33 of them the
// block's.  4096 x 4096 sites, C = 10, us per step at densities 36 and 360 (70
// steps after the first five): 456 and 441 before, 361 and 404 now; two sites per
// lane with 32-bit loads, and loads one tile ahead, gained nothing on it.  K[] packs the differences 2^7 - K_j
// (2^15 - K_j).  Adding r to each gives no carry, and its top bit is set
// exactly when K_j <= r: a count is an addition, a mask and a population
// count per word, where differences of 16-bit sums took three instructions
// of the slower kinds (packed 16-bit, 4.4 cycles a wave; additions and masks
// take 2.3).
template <int W>
__device__ __forceinline__ void collide_packed(uint32_t (&K)[W], const uint32_t *rules, uint32_t N,
                                               const Step9 &a, uint32_t s, uint32_t rid) {
  constexpr uint32_t kStride = W == 2 ? kRule9Byte : kRule9Half;
  constexpr uint32_t kRep = W == 2 ? 0u : 0x01000100u;  // byte (half) 0 in every place
  constexpr uint32_t kTop = W == 2 ? 0x80808080u : 0x80008000u;
  const SiteBlocks block(make_uint2((uint32_t)a.seed, (uint32_t)(a.seed >> 32)), s, (uint32_t)a.t, rid);
  uint32_t used = 0;
  for (int32_t sub = 0; sub < a.C; ++sub) {
    const uint4 w = block((uint32_t)sub);
    uint32_t r[3];
    draws<true>(r, w, N, a, s, rid, used);
    const uint32_t R1 = __builtin_amdgcn_perm(r[0], r[0], kRep), R2 = __builtin_amdgcn_perm(r[1], r[1], kRep);
    const uint32_t U = __builtin_amdgcn_perm(r[2], r[2], 0x01000100u);
    uint32_t v = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) v += __builtin_popcount((R1 + K[i]) & kTop);
    v += v << 3;
#pragma unroll
    for (int i = 0; i < W; ++i) v += __builtin_popcount((R2 + K[i]) & kTop);
    const uint32_t *const rec = rules + v * kStride;
    const uint2 c = *reinterpret_cast<const uint2 *>(rec);
    const uint32_t q = __builtin_popcount((U + c.x) & 0x80008000u) + __builtin_popcount((U + c.y) & 0x80008000u);
    const uint2 *const d = reinterpret_cast<const uint2 *>(rec + 2u + q * W);
    const uint2 d0 = d[0];
    K[0] += d0.x;
    K[1] += d0.y;
    if constexpr (W == 4) {
      const uint2 d1 = d[1];
      K[2] += d1.x;
      K[3] += d1.y;
    }
  }
}

// The same for any N and D, with the sums K_j as packed 16-bit pairs: the
// velocity of particle r is #{j : K_j <= r}, and a collision adds one of the
// rule table's packed changes.
__device__ __forceinline__ void collide_wide(u16x2 (&K)[4], const uint4 *rules, uint32_t N,
                                             const Step9 &a, uint32_t s, uint32_t rid) {
  uint32_t used = 0;
  uint32_t one_ = 0x10001u, one32_ = 1u;
  // opaque constants: no compare-and-select rewrite of the minima below
  asm volatile("" : "+v"(one_), "+v"(one32_));
  const u16x2 one = as_u16x2(one_);
  const SiteBlocks block(make_uint2((uint32_t)a.seed, (uint32_t)(a.seed >> 32)), s, (uint32_t)a.t, rid);
  for (int32_t sub = 0; sub < a.C; ++sub) {
    const uint4 w = block((uint32_t)sub);
    uint32_t r[3];
    draws<false>(r, w, N, a, s, rid, used);
    const uint32_t v1 = count_partial_le(K, r[0], one), v2 = count_partial_le(K, r[1], one);
    const uint32_t rec = (v1 * 9u + v2) * (kRule9Wide / 4);
    const uint4 c = rules[rec];
    // q = #{cumulative weights <= u} (u + 1 <= D < 2^32)
    const uint32_t u1 = r[2] + 1u, one32 = one32_;
    uint32_t q = __builtin_elementwise_min(__builtin_elementwise_sub_sat(u1, c.x), one32) +
                       __builtin_elementwise_min(__builtin_elementwise_sub_sat(u1, c.y), one32) +
                       __builtin_elementwise_min(__builtin_elementwise_sub_sat(u1, c.z), one32) +
                       __builtin_elementwise_min(__builtin_elementwise_sub_sat(u1, c.w), one32);
    asm volatile("" : "+v"(q));  // one shift for the record offset
    const uint4 d = rules[rec + 1u + q];
    K[0] += as_u16x2(d.x);
    K[1] += as_u16x2(d.y);
    K[2] += as_u16x2(d.z);
    K[3] += as_u16x2(d.w);
  }
}

// The table a block holds: 1 byte, 2 half, 3 wide; it only grows.  A wave's
// need goes to the place of its tile's parity, which nothing else reads or
// writes between two barriers; all waves of the block call this per tile.
constexpr uint32_t kRulesLds = rule9_words(kRule9Wide);
static_assert(kRulesLds >= rule9_words(kRule9Half) && kRulesLds >= rule9_words(kRule9Byte), "room for each table");
struct Table9 {
  const uint4 *src;
  uint32_t n;  // 16-byte pieces
};
__device__ __forceinline__ Table9 table9(const Step9 &a, uint32_t which) {
  const uint32_t at = which == 1u ? kRule9ByteAt : which == 2u ? kRule9HalfAt : kRule9WideAt;
  const uint32_t words = rule9_words(which == 1u ? kRule9Byte : which == 2u ? kRule9Half : kRule9Wide);
  return Table9{reinterpret_cast<const uint4 *>(a.rules + at), words / 4u};
}
__device__ __forceinline__ void hold_rules(const Step9 &a, uint32_t *rules, uint32_t *needs,
                                           uint32_t &held) {
  // (a barrier that waits for the LDS only: the last tile's stores stay in
  // flight)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  const uint32_t need = __builtin_amdgcn_readfirstlane(max(held, *needs));
  if (need == held) return;
  // (every wave's: it read the old table in an earlier tile, if at all)
  const Table9 tb = table9(a, need);
  for (uint32_t i = threadIdx.x; i < tb.n; i += blockDim.x) reinterpret_cast<uint4 *>(rules)[i] = tb.src[i];
  held = need;
  __syncthreads();
}

// The collisions of one site's counts n with the table the block holds.
__device__ __forceinline__ void collide_site(uint32_t (&n)[9], uint32_t N, const uint32_t *rules,
                                             uint32_t held, const Step9 &a, uint32_t s, uint32_t rid) {
  uint32_t K[8], k = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) K[j] = k += n[j];
  if (held == 1u) {
    uint32_t B[2];
#pragma unroll
    for (int m = 0; m < 2; ++m)
      B[m] = 0x80808080u - (K[4 * m] | K[4 * m + 1] << 8 | K[4 * m + 2] << 16 | K[4 * m + 3] << 24);
    collide_packed<2>(B, rules, N, a, s, rid);
#pragma unroll
    for (int j = 0; j < 8; ++j) K[j] = ((0x80808080u - B[j / 4]) >> (8 * (j & 3))) & 0xFFu;
  } else if (held == 2u) {
    uint32_t H[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) H[m] = 0x80008000u - (K[2 * m] | K[2 * m + 1] << 16);
    collide_packed<4>(H, rules, N, a, s, rid);
#pragma unroll
    for (int j = 0; j < 8; ++j) K[j] = ((0x80008000u - H[j / 2]) >> (16 * (j & 1))) & 0xFFFFu;
  } else {
    u16x2 P[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) P[m] = as_u16x2(K[2 * m] | K[2 * m + 1] << 16);
    collide_wide(P, reinterpret_cast<const uint4 *>(rules), N, a, s, rid);
#pragma unroll
    for (int j = 0; j < 8; ++j) K[j] = (as_u32(P[j / 2]) >> (16 * (j & 1))) & 0xFFFFu;
  }
#pragma unroll
  for (int j = 0; j < 9; ++j) n[j] = (j == 8 ? N : K[j]) - (j ? K[j - 1] : 0u);
}

// One step of every site: the literal loop of C sub-collisions (Eq. (select),
// Eq. (omega) with the D2Q9 rules), in place in the shifted layout.  Sites
// with N < 2 (or C = 0) are left untouched.  A block takes tiles of 256 sites
// in turn; it holds the rule table it began with until one of its sites needs a
// wider one.  Sub-collision k reads Philox block (s, t,
// replica, 2 | k << 2): words 0, 1, 2 draw the first particle, the second and
// the target.
__global__ void __launch_bounds__(kTileSites9) k_step9(Step9 a, uint32_t n_tiles) {
  __shared__ __align__(16) uint32_t rules[kRulesLds];
  __shared__ uint32_t needs[2];
  // (the table that most tiles need comes in beside the rest, not after the
  // first tile's counts: the steps of small lattices are a chain of latencies)
  const uint32_t first = a.first_table;
  uint32_t held = first, par = 0;
  const Table9 tb = table9(a, first);
  for (uint32_t i = threadIdx.x; i < tb.n; i += blockDim.x) reinterpret_cast<uint4 *>(rules)[i] = tb.src[i];
  if (threadIdx.x < 2u) needs[threadIdx.x] = first;
  __syncthreads();
  uint32_t rep = ~0u, tx = 0, ty = 0;
  Rep9 rp{};
  for (uint32_t it = blockIdx.x; it < n_tiles; it += gridDim.x, par ^= 1u) {
    const Tile9 tile = a.tiles[it];
    if (tile.rep != rep) {
      rep = tile.rep;
      rp = a.reps[rep];
      tx = a.no_stream ? 0u : (uint32_t)(a.t % rp.Lx);
      ty = a.no_stream ? 0u : (uint32_t)(a.t % rp.Ly);
    }
    bool act = tile.s0 + threadIdx.x < rp.S;
    // (lanes after the last site read its counts)
    const uint32_t i = act ? threadIdx.x : rp.S - 1u - tile.s0, s = tile.s0 + i;
    uint32_t x = tile.x0 + i;
    if (rp.Lx >= kTileSites9)  // a tile ends in its first row or the next
      x -= x >= rp.Lx ? rp.Lx : 0u;
    else
      x %= rp.Lx;
    const Site9 ph(s, x, tx, ty, rp.Lx, rp.S);
    uint32_t n[9], N = 0;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      n[j] = *at9(a.state, rp, j, ph.e[j]);
      N += n[j];
    }
    if (act && N > 65535u) atomicOr(a.err, kErrOverflow);
    act = act && N >= 2u && N <= 65535u;
    if (__ballot(act && N >= 0x80u) != 0u)
      atomicMax(&needs[par], __ballot(act && N >= 0x8000u) != 0u ? 3u : 2u);
    hold_rules(a, rules, &needs[par], held);
    if (!act) continue;
    collide_site(n, N, rules, held, a, s, rp.rid);
#pragma unroll
    for (int j = 0; j < 9; ++j) *at9(a.state, rp, j, ph.e[j]) = (uint16_t)n[j];
  }
}

// `steps` steps of lattices of up to 512 sites, one per block, a site per
// thread: the counts stay in LDS, in the same shifted layout, between one read
// and one write of the state.  Without the state's way through memory and a
// launch per step; bound by the latency of a wave's sub-collisions, two waves
// per SIMD.  Us per step: a lattice of 16 x 16 sites 5.7 with a launch each and
// 3.1 here, of 25 x 20 sites 6.2 and 3.9.  (With 1000 sites the 16 waves on one
// CU take 6.2, where four blocks of k_step9 take 5.9.)
__global__ void __launch_bounds__(kBlockSites9) k_steps9(Step9 a, uint32_t steps) {
  extern __shared__ __align__(16) uint16_t counts[];  // 9 arrays of S
  __shared__ __align__(16) uint32_t rules[kRulesLds];
  __shared__ uint32_t needs[2];
  const Rep9 rp = a.reps[blockIdx.x];
  const uint32_t S = rp.S, s = min(threadIdx.x, S - 1u), x = s % rp.Lx;
  for (uint32_t i = 0; i < 9u; ++i)
    for (uint32_t e = threadIdx.x; e < S; e += blockDim.x) counts[i * S + e] = *at9(a.state, rp, (int)i, e);
  uint32_t held = a.first_table;  // (see k_step9)
  const Table9 tb = table9(a, held);
  for (uint32_t i = threadIdx.x; i < tb.n; i += blockDim.x) reinterpret_cast<uint4 *>(rules)[i] = tb.src[i];
  if (threadIdx.x < 2u) needs[threadIdx.x] = held;
  uint32_t tx = a.no_stream ? 0u : (uint32_t)(a.t % rp.Lx), ty = a.no_stream ? 0u : (uint32_t)(a.t % rp.Ly);
  for (uint32_t k = 0; k < steps; ++k) {
    __syncthreads();  // the counts of this step are in place
    const Site9 ph(s, x, tx, ty, rp.Lx, S);
    uint32_t n[9], N = 0;
#pragma unroll
    for (int j = 0; j < 9; ++j) {
      n[j] = counts[(uint32_t)j * S + ph.e[j]];
      N += n[j];
    }
    bool act = threadIdx.x < S;
    if (act && N > 65535u) atomicOr(a.err, kErrOverflow);
    act = act && N >= 2u && N <= 65535u;
    if (__ballot(act && N >= 0x80u) != 0u)
      atomicMax(&needs[k & 1u], __ballot(act && N >= 0x8000u) != 0u ? 3u : 2u);
    hold_rules(a, rules, &needs[k & 1u], held);
    if (act) {
      collide_site(n, N, rules, held, a, s, rp.rid);
#pragma unroll
      for (int j = 0; j < 9; ++j) counts[(uint32_t)j * S + ph.e[j]] = (uint16_t)n[j];
    }
    ++a.t;
    if (!a.no_stream) {
      tx = tx + 1u == rp.Lx ? 0u : tx + 1u;
      ty = ty + 1u == rp.Ly ? 0u : ty + 1u;
    }
  }
  __syncthreads();
  for (uint32_t i = 0; i < 9u; ++i)
    for (uint32_t e = threadIdx.x; e < S; e += blockDim.x) *at9(a.state, rp, (int)i, e) = counts[i * S + e];
}

// Poisson start: site s draws Philox blocks (s, j, replica, 1), j = 0, 1, 2;
// word w of block j serves velocity 4 j + w.  At t = 0 the layout is
// unshifted.
__global__ void __launch_bounds__(256) k_init9_poisson(
    uint16_t *__restrict__ state, const Rep9 *__restrict__ reps, const Tile9 *__restrict__ tiles,
    const PoisDesc *__restrict__ desc, const uint32_t *__restrict__ pool, uint64_t seed,
    uint32_t *err) {
  const Tile9 tile = tiles[blockIdx.x];
  const Rep9 rp = reps[tile.rep];
  const uint32_t s = tile.s0 + threadIdx.x;
  if (s >= rp.S) return;
  const uint2 key = make_uint2((uint32_t)seed, (uint32_t)(seed >> 32));
#pragma unroll
  for (uint32_t j = 0; j < 3; ++j) {
    const uint4 w = philox10(make_uint4(s, j, rp.rid, 1u), key);
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      const uint32_t i = 4 * j + q;
      if (i >= 9) break;
      const PoisDesc d = desc[9u * tile.rep + i];
      const uint32_t n = d.k_first + count_le(pool + d.off, d.nthr, word_of(w, q));
      if (n > 65535u) atomicOr(err, kErrOverflow);
      state[rp.off + (uint64_t)i * rp.stride + s] = (uint16_t)n;
    }
  }
}

// Counts given in logical order ([9][Ly][Lx] per replica, replicas packed
// from dense[rep]); at t = 0 the layout is unshifted.  Counts the tiles that
// hold a site of 128 or more particles.
__global__ void __launch_bounds__(256) k_init9_counts(uint16_t *__restrict__ state,
                                                      const Rep9 *__restrict__ reps,
                                                      const Tile9 *__restrict__ tiles,
                                                      const uint64_t *__restrict__ dense,
                                                      const uint16_t *__restrict__ counts,
                                                      uint32_t *full) {
  const Tile9 tile = tiles[blockIdx.x];
  const Rep9 rp = reps[tile.rep];
  const uint32_t s = tile.s0 + threadIdx.x;
  uint32_t N = 0;
  if (s < rp.S) {
    const uint16_t *src = counts + dense[tile.rep];
#pragma unroll
    for (uint32_t i = 0; i < 9; ++i) {
      const uint16_t n = src[(uint64_t)i * rp.S + s];
      state[rp.off + (uint64_t)i * rp.stride + s] = n;
      N += n;
    }
  }
  if (__syncthreads_or(N >= 0x80u) && threadIdx.x == 0) atomicAdd(full, 1u);
}

// Occupation-number histograms of D2Q9 replicas, as k_histogram: each block
// takes a run of tiles, bins the nine arrays of their sites in LDS and adds
// the non-empty bins to its replica's row whenever the run changes replica.
__global__ void __launch_bounds__(256) k_histogram9(const uint16_t *__restrict__ state,
                                                    const Rep9 *__restrict__ reps,
                                                    const Tile9 *__restrict__ tiles,
                                                    uint32_t n_tiles, uint32_t n_bins,
                                                    unsigned long long *__restrict__ hist) {
  extern __shared__ uint32_t bins[];  // [9][n_bins]
  const uint32_t per = (n_tiles + gridDim.x - 1u) / gridDim.x;
  const uint32_t t_begin = blockIdx.x * per, t_end = min(n_tiles, t_begin + per);
  if (t_begin >= t_end) return;
  const uint32_t nb9 = 9u * n_bins, top = n_bins - 1u;
  for (uint32_t j = threadIdx.x; j < nb9; j += blockDim.x) bins[j] = 0u;
  uint32_t cur = tiles[t_begin].rep;
  auto flush = [&](uint32_t rep) {
    __syncthreads();
    unsigned long long *row = hist + (uint64_t)rep * nb9;
    for (uint32_t j = threadIdx.x; j < nb9; j += blockDim.x) {
      const uint32_t v = bins[j];
      if (v) {
        atomicAdd(&row[j], (unsigned long long)v);
        bins[j] = 0u;
      }
    }
    __syncthreads();
  };
  __syncthreads();
  for (uint32_t t = t_begin; t < t_end; ++t) {
    const Tile9 tile = tiles[t];
    if (tile.rep != cur) {
      flush(cur);
      cur = tile.rep;
    }
    const Rep9 rp = reps[tile.rep];
    const uint32_t s = tile.s0 + threadIdx.x;
    if (s < rp.S) {
#pragma unroll
      for (uint32_t i = 0; i < 9u; ++i) {
        const uint32_t n = state[rp.off + (uint64_t)i * rp.stride + s];
        atomicAdd(&bins[i * n_bins + min(n, top)], 1u);
      }
    }
  }
  flush(cur);
}

}  // namespace

hipError_t launch_step9(hipStream_t s, const Step9 &a, uint32_t n_tiles) {
  if (n_tiles == 0) return hipSuccess;  // (without sub-collisions a step still flags overflows)
  // Several tiles per block share a table; four times the blocks that fit the
  // chip even out their ends.  4096 x 4096 sites at density 36, us per step:
  // 2048 blocks 383, 8192 345, 32768 349, a block per tile 363.
  k_step9<<<std::min<uint32_t>(n_tiles, 8192u), kTileSites9, 0, s>>>(a, n_tiles);
  return hipGetLastError();
}

hipError_t launch_steps9(hipStream_t s, const Step9 &a, uint32_t n_reps, uint32_t max_sites,
                         uint32_t steps) {
  if (n_reps == 0 || steps == 0) return hipSuccess;
  if (max_sites > kBlockSites9) return hipErrorInvalidValue;
  k_steps9<<<n_reps, (max_sites + 63u) / 64u * 64u, 18u * max_sites, s>>>(a, steps);
  return hipGetLastError();
}

hipError_t launch_init9_poisson(hipStream_t s, uint16_t *state, const Rep9 *reps,
                                const Tile9 *tiles, uint32_t n_tiles, const PoisDesc *desc,
                                const uint32_t *pool, uint64_t seed, uint32_t *err) {
  if (n_tiles == 0) return hipSuccess;
  k_init9_poisson<<<n_tiles, 256, 0, s>>>(state, reps, tiles, desc, pool, seed, err);
  return hipGetLastError();
}

hipError_t launch_init9_counts(hipStream_t s, uint16_t *state, const Rep9 *reps,
                               const Tile9 *tiles, uint32_t n_tiles, const uint64_t *dense,
                               const uint16_t *counts, uint32_t *full) {
  if (n_tiles == 0) return hipSuccess;
  k_init9_counts<<<n_tiles, 256, 0, s>>>(state, reps, tiles, dense, counts, full);
  return hipGetLastError();
}

hipError_t launch_histogram9(hipStream_t s, const uint16_t *state, const Rep9 *reps,
                             const Tile9 *tiles, uint32_t n_tiles, uint32_t n_bins,
                             unsigned long long *hist) {
  if (n_tiles == 0) return hipSuccess;
  const uint32_t blocks = std::min<uint32_t>(n_tiles, 2048u);
  k_histogram9<<<blocks, 256, 9u * n_bins * sizeof(uint32_t), s>>>(state, reps, tiles, n_tiles,
                                                                   n_bins, hist);
  return hipGetLastError();
}

}  // namespace mclg
