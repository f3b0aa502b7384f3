// Step kernels that hold the sites they advance in registers (gfx950).
//
// A wave takes 64 x 4Q consecutive sites of one D1Q3 lattice into registers
// (a lane's 4Q sites as packed pairs of uint16 counts), advances them several
// steps there and writes them back once.  A step decides the collisions from
// the LDS image as the other step kernels do and then streams: n_+1 moves one
// site up and n_-1 one site down, a funnel shift per packed pair and one
// lane-to-lane move per array.  What bounds it is VALU issue (a step reads
// and writes no state), where the kernels that keep the state in memory are
// bound by the caches' bandwidth or, for small lattices, by a launch per step.
//
//   k_ring: a lattice that fits a block's registers, with its own periodic
//     boundary: the block's waves hold consecutive runs of sites and pass the
//     two counts that cross each wave boundary through LDS every step.
//   k_tile: any other lattice, cut into tiles.  A tile is held with kh sites
//     more on each side, whose values go wrong one site per step from the
//     ends, and is written back after at most kh steps.
#include "collide.h"
#include "device.h"
#include "mom3_sum.h"
#include "rng.h"

#include <algorithm>

namespace mclg {
namespace {

// The counts of a lane's 4Q consecutive sites.
template <int Q>
struct Sites {
  uint32_t m[2 * Q], z[2 * Q], p[2 * Q];
};

// The launch record in the kernel's argument segment.  What only undecided
// draws need (tables, parameters, the error word) is read through `cold()`,
// whose opaque pointer keeps those loads where they are used: hoisted out of
// the step loop they would take more scalar registers than there are.
typedef __attribute__((address_space(4))) const StepLaunch KernArgs;
__device__ __forceinline__ KernArgs *kernel_args() {
  return (KernArgs *)__builtin_amdgcn_kernarg_segment_ptr();
}

// What the steps of one lattice need besides the counts (wave-uniform but
// for `lane`).
struct Env {
  uint4 *queue;   // kQueue entries of LDS per wave
  uint2 key;
  LdsView lv;
  uint32_t Lp;    // positions of one period: the lattice's sites, rounded up to 8
  uint32_t rid, lane;
};

// Which of a wave's positions (site 0 of lane 0 first) count: positions from
// `end` on hold no sites (slow: some position of the wave is past it), and
// errors are flagged for positions own_lo <= pos < own_hi only.
struct Span {
  uint32_t end, own_lo, own_hi;
  bool slow;
};

// The random words of the NS sites from x on (x a multiple of 4, of 8 for
// eight sites; NS sites never pass the end of the period).
template <int NS>
__device__ __forceinline__ void draw_words(uint32_t (&r)[NS], uint32_t x, uint32_t t,
                                           const Env &E) {
  uint4 w0 = make_uint4(x >> 2, t, E.rid, 0u);
  if constexpr (NS == 4) {
    w0 = philox10(w0, E.key);
  } else {
    uint4 w1 = make_uint4((x >> 2) + 1u, t, E.rid, 0u);
    philox10_x2(w0, w1, E.key);
    r[4] = w1.x; r[5] = w1.y; r[6] = w1.z; r[7] = w1.w;
  }
  r[0] = w0.x; r[1] = w0.y; r[2] = w0.z; r[3] = w0.w;
}

__device__ __forceinline__ uint32_t fold16(uint32_t hi, uint32_t lo) {
  return __builtin_amdgcn_alignbit(hi, lo, 16);
}

// The launch's arguments, read where they are used.
__device__ __forceinline__ const void *kernel_args_now() {
  KernArgs *ka = kernel_args();
  asm volatile("" : "+s"(ka));
  return (const void *)ka;
}

// The exact outcome of one site as a move of its n_0 by -2 d.
template <bool GAL, bool MANY>
__device__ __forceinline__ uint32_t exact_move(const uint4 e, const Env &E, uint32_t t, bool own) {
  const StepLaunch *k = static_cast<const StepLaunch *>(kernel_args_now());
  const uint32_t bn = resolve_queued<GAL, MANY>(e, k->p, k->tab, t, E.rid, k->err, own);
  return (uint32_t)(((int32_t)(e.y >> 16) - (int32_t)bn) >> 1);
}

// Collisions of chunk C (the lane's sites 8C .. 8C + 7; Q = 1: its four
// sites), decided from the LDS image.  The sites it does not decide keep
// their counts; they go to the wave's queue (bit 8C + k of `und`: the lane's
// site 8C + k is in it; of `cols`: some lane's is; F entries so far), which
// is resolved at the end of the step.  A chunk with more such sites than the
// queue has room for only marks them (bit C of `dense`) for dense_chunks (Q = 6:
// it is left as it is, for dense_sites).
template <int Q, int C, bool FIXED>
__device__ __forceinline__ void collide_chunk(Sites<Q> &R, uint32_t &und, uint32_t &cols,
                                              uint32_t &dense, uint32_t &F, const Env &E,
                                              uint32_t x, uint32_t pos, const Span &S,
                                              uint32_t t) {
  constexpr int NS = Q == 1 ? 4 : 8, NP = NS / 2, W0 = 4 * C, K0 = 8 * C;
  uint32_t va[4], vb[4], vc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    va[j] = j < NP ? R.m[W0 + (j < NP ? j : 0)] : 0u;
    vb[j] = j < NP ? R.z[W0 + (j < NP ? j : 0)] : 0u;
    vc[j] = j < NP ? R.p[W0 + (j < NP ? j : 0)] : 0u;
  }
  uint32_t row[NS];
  u16x2 bi[NP];
  site_dir_pair<0>(row[0], row[1], bi[0], va, vb, vc, E.lv);
  site_dir_pair<1>(row[2], row[3], bi[1], va, vb, vc, E.lv);
  if constexpr (NS == 8) {
    site_dir_pair<2>(row[4], row[5], bi[2], va, vb, vc, E.lv);
    site_dir_pair<3>(row[6], row[7], bi[3], va, vb, vc, E.lv);
  }
  uint32_t r[NS];
  draw_words<NS>(r, x, t, E);
  SiteLook s[NS];
#pragma unroll
  for (int j = 0; j < NP; ++j) rec_pair(s[2 * j], s[2 * j + 1], row[2 * j], row[2 * j + 1], bi[j]);
  uint64_t mk[NS];  // the lanes whose site k is undecided
  uint32_t d[NP], n = 0;
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    d[j] = finish_pair<FIXED>(s[2 * j], s[2 * j + 1], r[2 * j], r[2 * j + 1], E.lv, mk[2 * j],
                             mk[2 * j + 1]);
  }
  if (S.slow) {
#pragma unroll
    for (int k = 0; k < NS; ++k) mk[k] &= lanes_gt(S.end, pos + k);
  }
#pragma unroll
  for (int k = 0; k < NS; ++k) n += (uint32_t)__popcll(mk[k]);
  if (n != 0u) {
    if (F + n > kQueue) {
      dense |= 1u << C;
#pragma unroll
      for (int j = 0; j < NP; ++j)
        if (Q == 6) d[j] = 0u;
#pragma unroll
      for (int k = 0; k < NS; ++k)
        if (Q != 6 && __builtin_amdgcn_inverse_ballot_w64(mk[k])) {
          d[k >> 1] &= (k & 1) ? 0x0000ffffu : 0xffff0000u;
          und |= 1u << (K0 + k);
        }
    } else {
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        if (mk[k] == 0) continue;
        if (__builtin_amdgcn_inverse_ballot_w64(mk[k])) {
          d[k >> 1] &= (k & 1) ? 0x0000ffffu : 0xffff0000u;
          und |= 1u << (K0 + k);
          const uint32_t wa = va[k >> 1], wb = vb[k >> 1], wc = vc[k >> 1];
          const uint32_t ab = (k & 1) ? __builtin_amdgcn_perm(wb, wa, 0x07060302u)
                                      : __builtin_amdgcn_perm(wb, wa, 0x05040100u);
          E.queue[F + lanes_below(mk[k])] =
              make_uint4(pos + k, ab, (k & 1) ? wc >> 16 : wc & 0xffffu, r[k]);
        }
        cols |= 1u << (K0 + k);
        F += (uint32_t)__popcll(mk[k]);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NP; ++j) apply_pair(R.m[W0 + j], R.z[W0 + j], R.p[W0 + j], d[j]);
}

// Resolves the queue's F entries exactly, lane i entry i; its move, in both
// halves, takes the place of entry i (word i of the queue's LDS).
template <bool GAL, bool MANY>
__device__ __forceinline__ void resolve_queue(uint32_t F, const Env &E, uint32_t xw, const Span &S,
                                              uint32_t t) {
  uint32_t *const res = reinterpret_cast<uint32_t *>(E.queue);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  uint32_t d2 = 0;
  if (E.lane < F) {
    uint4 e = E.queue[E.lane];
    const bool own = e.x >= S.own_lo && e.x < S.own_hi;
    e.x += xw;
    e.x -= e.x >= E.Lp ? E.Lp : 0u;
    d2 = (exact_move<GAL, MANY>(e, E, t, own) & 0xffffu) * 0x10001u;
  }
  __builtin_amdgcn_wave_barrier();  // every entry is read before a result is written over it
  res[E.lane] = d2;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The queued draws: resolved, then every lane takes the moves of its own
// sites back from the queue's LDS.  The queue is empty again.
template <int Q, bool GAL>
__device__ __forceinline__ void resolve_step(Sites<Q> &R, uint32_t &und, uint32_t &cols, uint32_t &F,
                                             const Env &E, uint32_t xw, const Span &S,
                                             uint32_t t) {
  uint32_t *const res = reinterpret_cast<uint32_t *>(E.queue);
  resolve_queue<GAL, false>(F, E, xw, S, t);
  uint32_t base = 0;
#pragma unroll
  for (int k = 0; k < 4 * Q; ++k) {
    if (!(cols & (1u << k))) continue;
    const bool mine = (und & (1u << k)) != 0u;
    const uint64_t mk = __ballot(mine);
    const uint32_t v = res[(base + lanes_below(mk)) & (kQueue - 1u)];
    const uint32_t d = mine ? v & ((k & 1) ? 0xffff0000u : 0x0000ffffu) : 0u;
    apply_pair(R.m[k >> 1], R.z[k >> 1], R.p[k >> 1], d);
    base += (uint32_t)__popcll(mk);
  }
  und &= ~cols;
  F = cols = 0u;
  // the results are read before the next entries are written
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The undecided sites of the chunks in `dense`, in batches of up to 64 that
// go through the queue.  An iteration of the outer loop handles the lane's
// first four sites, drawn anew, and rotates its words by four sites, so the
// registers are fixed and the code is short.  Its cost goes with the number
// of undecided sites: 2^24 sites of density 100 and mean velocity 0.2, where
// 12 % are, took 72 us per step with a batch per site of a lane (every site
// of such a chunk) and take 45
// (Q = 4).
template <int Q, bool GAL>
__device__ __forceinline__ void dense_chunks(Sites<Q> &R, uint32_t dense, uint32_t und, const Env &E,
                                             uint32_t x, uint32_t pos, uint32_t xw, const Span &S,
                                             uint32_t t) {
  constexpr int W = 2 * Q;
  const uint32_t *const res = reinterpret_cast<const uint32_t *>(E.queue);
#pragma unroll 1
  for (uint32_t q = 0; q < (uint32_t)Q; ++q) {
    if (dense & (1u << (q >> 1))) {
      uint32_t r[4], at[4], d[2] = {0u, 0u}, n = 0;
      draw_words<4>(r, x, t, E);
      // the sites without a row first: their sub-collisions one by one take
      // many times what a row does, for a whole batch
      const uint32_t n_max = static_cast<const StepLaunch *>(kernel_args_now())->p.n_max;
      uint32_t lit = 0;
#pragma unroll
      for (uint32_t k = 0; k < 4u; ++k) {
        const uint32_t sh = 16u * (k & 1u);
        const uint32_t N = ((R.m[k >> 1] >> sh) & 0xffffu) + ((R.z[k >> 1] >> sh) & 0xffffu) +
                           ((R.p[k >> 1] >> sh) & 0xffffu);
        lit |= N > n_max ? und & (1u << k) : 0u;
        at[k] = ~0u;
      }
      auto number = [&](uint32_t which) {  // the sites' places among the undecided
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
          const bool mine = (which & (1u << k)) != 0u;
          const uint64_t mk = __ballot(mine);
          at[k] = mine ? n + lanes_below(mk) : at[k];
          n += (uint32_t)__popcll(mk);
        }
      };
      if (__ballot(lit != 0u) != 0u) number(lit);
      number(und & ~lit);
#pragma unroll 1
      for (uint32_t b0 = 0; b0 < n; b0 += kQueue) {
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
          const uint32_t wa = R.m[k >> 1], wb = R.z[k >> 1], wc = R.p[k >> 1];
          if (at[k] - b0 < kQueue)
            E.queue[at[k] - b0] =
                make_uint4(pos + k, __builtin_amdgcn_perm(wb, wa, (k & 1u) ? 0x07060302u : 0x05040100u),
                           (k & 1u) ? wc >> 16 : wc & 0xffffu, r[k]);
        }
        resolve_queue<GAL, true>(min(n - b0, kQueue), E, xw, S, t);
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k)
          if (at[k] - b0 < kQueue)
            d[k >> 1] |= res[at[k] - b0] & ((k & 1u) ? 0xffff0000u : 0x0000ffffu);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      apply_pair(R.m[0], R.z[0], R.p[0], d[0]);
      apply_pair(R.m[1], R.z[1], R.p[1], d[1]);
    }
    und >>= 4;
    x += 4u;
    x -= x >= E.Lp ? E.Lp : 0u;
    pos += 4u;
    if constexpr (W > 2) {
      const uint32_t m0 = R.m[0], m1 = R.m[1], z0 = R.z[0], z1 = R.z[1], p0 = R.p[0], p1 = R.p[1];
#pragma unroll
      for (int j = 0; j + 2 < W; ++j) {
        R.m[j] = R.m[j + 2];
        R.z[j] = R.z[j + 2];
        R.p[j] = R.p[j + 2];
      }
      R.m[W - 2] = m0; R.m[W - 1] = m1;
      R.z[W - 2] = z0; R.z[W - 1] = z1;
      R.p[W - 2] = p0; R.p[W - 1] = p1;
    }
  }
}

// The same for Q = 6, every site of the chunks from the global rows, each lane
// its own (batches need the registers that six times four sites take: at
// density 50, which has no such chunks, 28.5 us per step of 2^24 sites
// instead of 25.7; plan_ways keeps lattices with many of them from Q = 6).  An iteration of the outer loop handles
// the lane's first four sites and rotates its words by four sites, one of
// the inner loop the first site of those, so the registers are fixed and the
// code is short.
template <int Q, bool GAL>
__device__ __forceinline__ void dense_sites(Sites<Q> &R, uint32_t dense, const Env &E, uint32_t x,
                                             uint32_t pos, const Span &S, uint32_t t) {
  constexpr int W = 2 * Q;
#pragma unroll 1
  for (uint32_t q = 0; q < (uint32_t)Q; ++q) {
    if (dense & (1u << (q >> 1))) {
      uint32_t r[4];
      draw_words<4>(r, x, t, E);
#pragma unroll 1
      for (uint32_t k = 0; k < 4u; ++k) {
        const uint32_t at = pos + k;
        uint32_t d = 0;
        if (!S.slow || at < S.end)
          d = exact_move<GAL, true>(make_uint4(x + k, __builtin_amdgcn_perm(R.z[0], R.m[0], 0x05040100u),
                                         R.p[0] & 0xffffu, r[0]),
                              E, t, at >= S.own_lo && at < S.own_hi) & 0xffffu;
        apply_pair(R.m[0], R.z[0], R.p[0], d);
        uint32_t w;
        w = R.m[0]; R.m[0] = fold16(R.m[1], w); R.m[1] = fold16(w, R.m[1]);
        w = R.z[0]; R.z[0] = fold16(R.z[1], w); R.z[1] = fold16(w, R.z[1]);
        w = R.p[0]; R.p[0] = fold16(R.p[1], w); R.p[1] = fold16(w, R.p[1]);
        w = r[0]; r[0] = r[1]; r[1] = r[2]; r[2] = r[3]; r[3] = w;
      }
    }
    x += 4u;
    x -= x >= E.Lp ? E.Lp : 0u;
    pos += 4u;
    if constexpr (W > 2) {
      const uint32_t m0 = R.m[0], m1 = R.m[1], z0 = R.z[0], z1 = R.z[1], p0 = R.p[0], p1 = R.p[1];
#pragma unroll
      for (int j = 0; j + 2 < W; ++j) {
        R.m[j] = R.m[j + 2];
        R.z[j] = R.z[j + 2];
        R.p[j] = R.p[j + 2];
      }
      R.m[W - 2] = m0; R.m[W - 1] = m1;
      R.z[W - 2] = z0; R.z[W - 1] = z1;
      R.p[W - 2] = p0; R.p[W - 1] = p1;
    }
  }
}

// Without collisions a step only flags sites whose N does not fit 16 bits.
template <int Q>
__device__ __forceinline__ void flag_saturated(const Sites<Q> &R, const Env &E, uint32_t pos,
                                               const Span &S) {
  bool over = false;
#pragma unroll
  for (int j = 0; j < 2 * Q; ++j) {
    const uint32_t N2 = __builtin_bit_cast(
        uint32_t, __builtin_elementwise_add_sat(
                      __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, R.m[j]),
                                                    __builtin_bit_cast(u16x2, R.z[j])),
                      __builtin_bit_cast(u16x2, R.p[j])));
    const uint32_t a = pos + 2 * j;
    // (a saturated sum may be exactly 65535, which fits)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (((N2 >> (16 * h)) & 0xffffu) != 0xffffu) continue;
      const uint32_t N = ((R.m[j] >> (16 * h)) & 0xffffu) + ((R.z[j] >> (16 * h)) & 0xffffu) +
                         ((R.p[j] >> (16 * h)) & 0xffffu);
      over |= N > 65535u && a + h >= S.own_lo && a + h < S.own_hi;
    }
  }
  if (over) {
    KernArgs *ka = kernel_args();
    atomicOr(ka->err, kErrOverflow);
  }
}

constexpr uint32_t kFlushAt = 28;
// One step's collisions of the wave's sites; xw: the lattice site at
// position 0 (below L).
template <int Q, bool GAL, bool FIXED>
__device__ __forceinline__ void collide(Sites<Q> &R, const Env &E, uint32_t xw, const Span &S,
                                        uint32_t t, bool collisions) {
  uint32_t pos = E.lane * (4u * Q);
  // computed anew at every step: what the compiler would hoist out of the
  // step loop (positions, sites and first Philox products of every chunk)
  // takes more registers than it saves instructions
  asm volatile("" : "+v"(pos));
  if (!collisions) {
    flag_saturated<Q>(R, E, pos, S);
    return;
  }
  uint32_t F = 0, und = 0, cols = 0, dense = 0;
  auto at = [&](uint32_t o) {
    const uint32_t y = xw + pos + o;
    return y >= E.Lp ? y - E.Lp : y;
  };
  collide_chunk<Q, 0, FIXED>(R, und, cols, dense, F, E, at(0u), pos, S, t);
  // Emptied early where the next chunk's would not fit with these (Q = 6: see
  // dense_sites).
  if constexpr (Q >= 4) {
    if (Q == 4 && F > kFlushAt) resolve_step<Q, GAL>(R, und, cols, F, E, xw, S, t);
    collide_chunk<Q, 1, FIXED>(R, und, cols, dense, F, E, at(8u), pos + 8u, S, t);
  }
  if constexpr (Q >= 6) {
    collide_chunk<Q, 2, FIXED>(R, und, cols, dense, F, E, at(16u), pos + 16u, S, t);
  }
  if (F) resolve_step<Q, GAL>(R, und, cols, F, E, xw, S, t);
  if (dense) {
    if constexpr (Q == 6) dense_sites<Q, GAL>(R, dense, E, at(0u), pos, S, t);
    else dense_chunks<Q, GAL>(R, dense, und, E, at(0u), pos, xw, S, t);
  }
}

constexpr int kDppShl1 = 0x130, kDppRol1 = 0x134;  // lane i takes lane i + 1 (rol: 63 takes 0)
constexpr int kDppShr1 = 0x138, kDppRor1 = 0x13c;  // lane i takes lane i - 1 (ror: 0 takes 63)
// Streaming: n_+1 one site up, n_-1 one site down.  up_in: the count that
// enters at the first site (in the high half); down_in: the one that enters
// after the last site (in the low half); with ROT the wave's own.
template <int Q, bool ROT>
__device__ __forceinline__ void stream(Sites<Q> &R, uint32_t up_in, uint32_t down_in) {
  constexpr int W = 2 * Q;
  const uint32_t pi = (uint32_t)__builtin_amdgcn_update_dpp(
      (int)up_in, (int)R.p[W - 1], ROT ? kDppRor1 : kDppShr1, 0xf, 0xf, false);
#pragma unroll
  for (int j = W - 1; j > 0; --j) R.p[j] = fold16(R.p[j], R.p[j - 1]);
  R.p[0] = fold16(R.p[0], pi);
  const uint32_t mi = (uint32_t)__builtin_amdgcn_update_dpp(
      (int)down_in, (int)R.m[0], ROT ? kDppRol1 : kDppShl1, 0xf, 0xf, false);
#pragma unroll
  for (int j = 0; j + 1 < W; ++j) R.m[j] = fold16(R.m[j + 1], R.m[j]);
  R.m[W - 1] = fold16(mi, R.m[W - 1]);
}

// The count at position `pos` (wave-uniform) of one array, and its
// replacement.
template <int Q>
__device__ __forceinline__ uint32_t site_of(const uint32_t (&v)[2 * Q], uint32_t pos) {
  const uint32_t l = pos / (4u * Q), e = pos % (4u * Q);
  uint32_t w = 0;
#pragma unroll
  for (uint32_t j = 0; j < 2 * Q; ++j) {
    const uint32_t x = __builtin_amdgcn_readlane(v[j], l);
    w = (e >> 1) == j ? x : w;
  }
  return (e & 1u) ? w >> 16 : w & 0xffffu;
}
template <int Q>
__device__ __forceinline__ void set_site(uint32_t (&v)[2 * Q], uint32_t pos, uint32_t lane,
                                         uint32_t n) {
  const uint32_t l = pos / (4u * Q), e = pos % (4u * Q);
#pragma unroll
  for (uint32_t j = 0; j < 2 * Q; ++j)
    if ((e >> 1) == j && lane == l)
      v[j] = (e & 1u) ? (v[j] & 0xffffu) | n << 16 : (v[j] & 0xffff0000u) | n;
}

// Where a slot's arrays are.
struct Mem {
  Rsrc rs;
  uint32_t ab;  // bytes per array
  uint32_t L;
};
__device__ __forceinline__ Mem slot_mem(uint16_t *state, const SlotDev &sl) {
  Mem M;
  const uint64_t base = reinterpret_cast<uint64_t>(state + sl.off);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
  M.ab = __builtin_amdgcn_readfirstlane(2u * sl.stride);
  M.rs = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(((uint64_t)hi << 32) | lo), 0,
                                           (int)(3u * M.ab), kRsrcWord3);
  M.L = __builtin_amdgcn_readfirstlane(sl.L);
  return M;
}

// NS consecutive elements of an array, one vector access.
template <int NS>
__device__ __forceinline__ void vload(Rsrc r, uint32_t voff, uint32_t soff, uint32_t *v) {
  if constexpr (NS == 8) {
    const auto q = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0);
    v[0] = q[0]; v[1] = q[1]; v[2] = q[2]; v[3] = q[3];
  } else {
    const auto q = __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0);
    v[0] = q[0]; v[1] = q[1];
  }
}
template <int NS>
__device__ __forceinline__ void vstore(Rsrc r, uint32_t voff, uint32_t soff, const uint32_t *v) {
  if constexpr (NS == 8) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 q = {v[0], v[1], v[2], v[3]};
    __builtin_amdgcn_raw_buffer_store_b128(q, r, (int)voff, (int)soff, 0);
  } else {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 q = {v[0], v[1]};
    __builtin_amdgcn_raw_buffer_store_b64(q, r, (int)voff, (int)soff, 0);
  }
}
__device__ __forceinline__ void put16(uint32_t *w, int e, uint32_t v) {
  if (e & 1) w[e >> 1] = (w[e >> 1] & 0xffffu) | (v << 16);
  else w[e >> 1] = (w[e >> 1] & 0xffff0000u) | (v & 0xffffu);
}

// The NS sites from x on of a slot at shift tm (x < L; sites past L wrap when
// `wrap`, else the first `n` exist and the others read as empty).
template <int NS>
__device__ __forceinline__ void load_sites(const Mem &M, uint32_t x, uint32_t tm, bool wrap,
                                           uint32_t n, uint32_t *m, uint32_t *z, uint32_t *p) {
  uint32_t pm = x + tm;
  pm -= pm >= M.L ? M.L : 0u;
  const uint32_t pp = x >= tm ? x - tm : x + M.L - tm;
  if (x + NS <= M.L && pm + NS <= M.L && pp + NS <= M.L && n >= NS) {
    vload<NS>(M.rs, 2u * pm, 0u, m);
    vload<NS>(M.rs, 2u * x, M.ab, z);
    vload<NS>(M.rs, 2u * pp, 2u * M.ab, p);
    return;
  }
#pragma unroll
  for (int e = 0; e < NS; ++e) {
    uint32_t y = x + (uint32_t)e, va = 0, vb = 0, vc = 0;
    if ((uint32_t)e < n && (wrap || y < M.L)) {
      y -= y >= M.L ? M.L : 0u;
      uint32_t ym = y + tm;
      ym -= ym >= M.L ? M.L : 0u;
      const uint32_t yp = y >= tm ? y - tm : y + M.L - tm;
      va = bload2(M.rs, 2u * ym, 0u);
      vb = bload2(M.rs, 2u * y, M.ab);
      vc = bload2(M.rs, 2u * yp, 2u * M.ab);
    }
    put16(m, e, va); put16(z, e, vb); put16(p, e, vc);
  }
}
// The first n (<= NS) sites from x on (x + n <= L) back at shift tm.
template <int NS>
__device__ __forceinline__ void store_sites(const Mem &M, uint32_t x, uint32_t tm, uint32_t n,
                                            const uint32_t *m, const uint32_t *z,
                                            const uint32_t *p) {
  uint32_t pm = x + tm;
  pm -= pm >= M.L ? M.L : 0u;
  const uint32_t pp = x >= tm ? x - tm : x + M.L - tm;
  if (n >= NS && pm + NS <= M.L && pp + NS <= M.L) {
    vstore<NS>(M.rs, 2u * pm, 0u, m);
    vstore<NS>(M.rs, 2u * x, M.ab, z);
    vstore<NS>(M.rs, 2u * pp, 2u * M.ab, p);
    return;
  }
#pragma unroll
  for (int e = 0; e < NS; ++e) {
    if ((uint32_t)e < n) {
      const uint32_t y = x + (uint32_t)e;
      uint32_t ym = y + tm;
      ym -= ym >= M.L ? M.L : 0u;
      const uint32_t yp = y >= tm ? y - tm : y + M.L - tm;
      bstore2(M.rs, 2u * ym, 0u, (m[e >> 1] >> (16 * (e & 1))) & 0xffffu);
      bstore2(M.rs, 2u * y, M.ab, (z[e >> 1] >> (16 * (e & 1))) & 0xffffu);
      bstore2(M.rs, 2u * yp, 2u * M.ab, (p[e >> 1] >> (16 * (e & 1))) & 0xffffu);
    }
  }
}

// A slot's collision image into the block's LDS (from address 0).
__device__ __forceinline__ void copy_image(uint4 *lds, const uint8_t *pool, const ImageDesc &im) {
  const uint4 *src = reinterpret_cast<const uint4 *>(pool + im.off);
  const uint32_t n16 = im.bytes / 16u, bd = blockDim.x, last = n16 - 1u;
  // ten loads in flight per thread, then their stores
  for (uint32_t b0 = threadIdx.x; b0 < n16; b0 += 10u * bd) {
    uint4 v[10];
#pragma unroll
    for (uint32_t j = 0; j < 10; ++j) v[j] = src[min(b0 + j * bd, last)];
#pragma unroll
    for (uint32_t j = 0; j < 10; ++j)
      asm volatile("" : "+v"(v[j].x), "+v"(v[j].y), "+v"(v[j].z), "+v"(v[j].w));
#pragma unroll
    for (uint32_t j = 0; j < 10; ++j)
      if (b0 + j * bd < n16) lds[b0 + j * bd] = v[j];
  }
}
// ---------------------------------------------------------------------------
// Moments of the sites a wave holds
// ---------------------------------------------------------------------------
// The second argument of the kernels, in the kernel's argument segment: what
// a log needs is read where it is used (see kernel_args).
template <class Launch>
__device__ __forceinline__ const RegLog *log_args() {
  constexpr size_t at = (sizeof(StepLaunch) + alignof(Launch) - 1) / alignof(Launch) * alignof(Launch);
  const char *k = (const char *)kernel_args();
  asm volatile("" : "+s"(k));
  return reinterpret_cast<const RegLog *>(k + at + offsetof(Launch, log));
}

// Adds the moments of the wave's own sites (record slots as in moments.h) to
// `rec`, the wave's record of this log, or stores them there (`fresh`).
// The sums take the lane's words one pair of sites at a time, rotating them,
// so that a log in the middle of the steps needs few registers.
template <int Q>
__device__ __attribute__((noinline)) void log_sites(Sites<Q> R, uint32_t xw, uint32_t Lp, uint32_t L,
                                                    uint32_t own_lo, uint32_t own_hi,
                                                    const RegLog *lg, const int32_t *tw,
                                                    unsigned long long *rec, bool fresh) {
  const uint32_t lane = threadIdx.x & 63u;
  using namespace mom3;
  constexpr int W = 2 * Q;
  uint32_t pos = lane * (4u * Q);
  asm volatile("" : "+v"(pos));
  uint32_t x0 = xw + pos;
  x0 -= x0 >= Lp ? Lp : 0u;
  const uint32_t n_modes = lg->n_modes;
  const bool dig = lg->digest != 0u;
  {
    uint32_t s0 = 0, s1 = 0, s2 = 0, odd = 0, mx = 0;
    u64 q[6] = {}, d = 0;
    uint32_t at = pos, x = x0;
#pragma unroll 1
    for (int j = 0; j < W; ++j) {
#pragma unroll
      for (uint32_t h = 0; h < 2u; ++h) {
        const bool own = at + h >= own_lo && at + h < own_hi;
        const uint32_t a = own ? (R.m[0] >> (16u * h)) & 0xffffu : 0u;
        const uint32_t b = own ? (R.z[0] >> (16u * h)) & 0xffffu : 0u;
        const uint32_t c = own ? (R.p[0] >> (16u * h)) & 0xffffu : 0u;
        s0 += a;
        s1 += b;
        s2 += c;
        q[0] += (u64)a * a;
        q[1] += (u64)b * b;
        q[2] += (u64)c * c;
        q[3] += (u64)a * b;
        q[4] += (u64)b * c;
        q[5] += (u64)a * c;
        odd += b & 1u;
        mx = max(mx, a + b + c);
        if (dig) {
          const uint32_t k = 4u * (x + h) + 1u;
          if (own)
            d += (u64)fmix32(fmix32(k) ^ a) + fmix32(fmix32(k + 1u) ^ b) + fmix32(fmix32(k + 2u) ^ c);
        }
      }
      at += 2u;
      x += 2u;
      x -= x >= Lp ? Lp : 0u;
      const uint32_t fm = R.m[0], fz = R.z[0], fp = R.p[0];
#pragma unroll
      for (int i = 0; i + 1 < W; ++i) {
        R.m[i] = R.m[i + 1];
        R.z[i] = R.z[i + 1];
        R.p[i] = R.p[i + 1];
      }
      R.m[W - 1] = fm;
      R.z[W - 1] = fz;
      R.p[W - 1] = fp;
    }
    u64 v[16] = {s0, s1, s2, q[0], q[1], q[2], q[3], q[4], q[5], odd, d, 0, 0, 0, 0, 0};
    mx = wave_max(mx);
    u64 s = wave_sum_scatter<16>(v, lane);  // lane l: value l / 4
    const uint32_t slot = lane >> 2;
    if ((lane & 3u) == 0u && slot < 12u) {
      if (slot == 11u) s = mx;
      if (!fresh) {
        const u64 before = rec[slot];
        s = slot == 11u ? max(s, before) : s + before;
      }
      rec[slot] = s;
    }
  }
  // Fourier sums, one row of the twiddles at a time
#pragma unroll 1
  for (uint32_t m = 0; m < 2u * n_modes; ++m) {
    const int32_t *const row = tw + (uint64_t)m * L;
    int32_t w[4 * Q];
#pragma unroll
    for (int g = 0; g < Q; ++g) {
      uint32_t x = x0 + 4u * g;
      x -= x >= Lp ? Lp : 0u;
      if (x + 4u <= L) {
        __builtin_memcpy(&w[4 * g], row + x, 16);  // (4-byte aligned)
      } else {
#pragma unroll
        for (uint32_t e = 0; e < 4u; ++e) w[4 * g + e] = x + e < L ? row[x + e] : 0;
      }
    }
    i64 f = 0;
#pragma unroll
    for (int k = 0; k < 4 * Q; ++k) {
      const uint32_t sh = 16u * (k & 1);
      const uint32_t N = ((R.m[k >> 1] >> sh) & 0xffffu) + ((R.z[k >> 1] >> sh) & 0xffffu) +
                         ((R.p[k >> 1] >> sh) & 0xffffu);
      const bool own = pos + k >= own_lo && pos + k < own_hi;
      f += (i64)(int32_t)(own ? N : 0u) * (i64)w[k];
    }
    u64 fs = (u64)f;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) fs += shfl_xor_u64(fs, o);
    if (lane == 0u) rec[12u + m] = fresh ? fs : rec[12u + m] + fs;
  }
}

// The results of a launch's logs from the waves' records: block (j, u) adds
// the `held` records of lattice u (of `stride`) at log j into its row.  Bound
// by the latency of its loads, eight in flight per thread: the 4096 records
// of a tile launch take 19 us (140 with one at a time in 256 threads).
__global__ void __launch_bounds__(1024) k_log_final(StepLaunch a, RegLog lg, const uint32_t *order,
                                                    uint32_t n, uint32_t t_off) {
  using namespace mom3;
  const uint32_t j = blockIdx.x / n, u = blockIdx.x % n, slot = order[u];
  const SlotDev sl = a.slots[slot];
  const unsigned long long *const rec = lg.records + ((uint64_t)j * n + u) * lg.stride * kMom3Rec;
  __shared__ u64 part[32][kMom3Rec];
  __shared__ u64 T[kMom3Rec];
  // thread (g, k): value k of records g, g + G, ...
  const uint32_t k = threadIdx.x & 31u, g = threadIdx.x >> 5, G = blockDim.x >> 5;
  const uint32_t hold = lg.hold ? (sl.L + lg.hold - 1u) / lg.hold : lg.stride;
  u64 s = 0;
  if (k < 12u + 2u * lg.n_modes)
    for (uint32_t w = g; w < hold; w += 8u * G) {
      u64 y[8];
#pragma unroll
      for (uint32_t i = 0; i < 8u; ++i)
        y[i] = w + i * G < hold ? rec[(uint64_t)(w + i * G) * kMom3Rec + k] : 0ull;
#pragma unroll
      for (uint32_t i = 0; i < 8u; ++i) s = k == 11u ? max(s, y[i]) : s + y[i];
    }
  part[g][k] = s;
  __syncthreads();
  if (threadIdx.x < kMom3Rec) {
    s = part[0][k];
    for (uint32_t i = 1; i < G; ++i) s = k == 11u ? max(s, part[i][k]) : s + part[i][k];
    T[k] = s;
  }
  __syncthreads();
  if (threadIdx.x < kMom3Out)
    lg.out[((uint64_t)j * a.n_slots + slot) * kMom3Out + threadIdx.x] = (i64)result_field(
        threadIdx.x, T, a.tslot[slot] + t_off + lg.first + j * lg.every, sl.L, lg.n_modes);
}

// ---------------------------------------------------------------------------
// Lattices that fit a block's registers
// ---------------------------------------------------------------------------
// rl.team = 0: the block holds one lattice, order[b], over as many of its
// waves as it needs.  rl.team = k > 0: each of the block's first k waves holds
// one, order[b k + wave], all with the same image.  The other waves only help
// to copy the image.
template <int Q, bool GAL, bool FIXED, bool LOG>
__global__ void __launch_bounds__(1024) k_ring(StepLaunch a, RingLaunch rl) {
  constexpr uint32_t S = 4u * Q, W = 2 * Q, NS = Q == 1 ? 4 : 8, NC = S / NS;
  extern __shared__ uint4 lds[];
  const uint32_t lane = threadIdx.x & 63u, nw = blockDim.x >> 6;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t u0 = rl.team ? blockIdx.x * rl.team : blockIdx.x;
  const uint32_t u = rl.team ? u0 + wave : u0;
  const uint32_t w = rl.team ? 0u : wave;
  const bool mine = rl.team ? wave < rl.team && u < rl.n : true;
  const uint32_t slot = __builtin_amdgcn_readfirstlane(rl.order[mine ? u : u0]);
  const ImageDesc im = a.images[slot];
  const SlotDev sl = a.slots[slot];
  const Mem M = slot_mem(a.state, sl);
  const uint32_t L = M.L;
  const uint32_t steps = __builtin_amdgcn_readfirstlane(rl.limit ? rl.limit[slot] : rl.steps);
  const uint32_t t0 = __builtin_amdgcn_readfirstlane(a.tslot[slot] + a.t_off);
  const uint32_t first = w * 64u * S;               // the wave's first site
  const uint32_t held = (L + 64u * S - 1u) / (64u * S);  // waves that hold the lattice
  const bool active = mine && w < held;             // (wave-uniform)
  const uint32_t x = first + lane * S;
  const bool ns = a.p.no_stream != 0u, coll = a.p.C != 0;
  Sites<Q> R;
#pragma unroll
  for (uint32_t j = 0; j < W; ++j) R.m[j] = R.z[j] = R.p[j] = 0u;
  if (active) {
    const uint32_t tm = ns ? 0u : t0 % L;
#pragma unroll
    for (uint32_t c = 0; c < NC; ++c) {
      const uint32_t xc = x + NS * c;
      if (xc < L)
        load_sites<NS>(M, xc, tm, false, NS, R.m + c * NS / 2, R.z + c * NS / 2, R.p + c * NS / 2);
    }
  }
  copy_image(lds, a.image_pool, im);
  const Env E{lds + a.lds_bytes / 16u + wave * (kWaveLdsBytes / 16u),
              make_uint2((uint32_t)a.p.seed, (uint32_t)(a.p.seed >> 32)), image_view(im), (L + 7u) & ~7u, sl.rid, lane};
  // the counts that cross wave boundaries, two buffers
  uint32_t *const xch = reinterpret_cast<uint32_t *>(lds + a.lds_bytes / 16u + nw * (kWaveLdsBytes / 16u));
  __syncthreads();  // the image is in place
  if (!active && held == 1u) return;  // no barrier below
  Span Sp;
  Sp.end = active ? L - first : 0u;
  Sp.own_lo = 0u;
  Sp.own_hi = 0xffffffffu;
  Sp.slow = first + 64u * S > L;
  // the wave's last site: its lane and element
  const uint32_t e1 = active ? min(L - first, 64u * S) - 1u : 64u * S - 1u;
  const uint32_t le = e1 / S, ee = e1 % S;
  uint32_t ins[W];  // the bits of that element in its lane's words
#pragma unroll
  for (uint32_t j = 0; j < W; ++j)
    ins[j] = (lane == le && (ee >> 1) == j) ? ((ee & 1u) ? 0xffff0000u : 0x0000ffffu) : 0u;
  uint32_t next = LOG ? rl.log.first : 0u, logs = 0;
  auto log = [&]() {  // the moments of the state the steps so far reach
    if (active) {
      const RegLog *lg = log_args<RingLaunch>();
      log_sites<Q>(R, first, E.Lp, L, 0u, Sp.end, lg, lg->tw + 2ull * lg->n_modes * sl.dense,
                   lg->records + (((uint64_t)logs * rl.n + u) * lg->stride + w) * kMom3Rec, true);
    }
    ++logs;
    next = logs < rl.log.n ? next + rl.log.every : 0u;
  };
  for (uint32_t s = 0; s < steps; ++s) {
    if (active) collide<Q, GAL, FIXED>(R, E, first, Sp, t0 + s, coll);
    if (ns) {
      if (LOG && s + 1u == next) log();
      continue;
    }
    uint32_t pl = site_of<Q>(R.p, e1);
    uint32_t mf = __builtin_amdgcn_readfirstlane(R.m[0]) & 0xffffu;
    if (held > 1u) {
      uint32_t *const b = xch + (s & 1u) * 16u;
      if (lane == 0) b[wave] = pl | mf << 16;
      __syncthreads();
      pl = b[w == 0u ? held - 1u : w - 1u] & 0xffffu;
      mf = b[w + 1u >= held ? 0u : w + 1u] >> 16;
    }
    stream<Q, false>(R, pl << 16, 0u);
    const uint32_t mv = mf * 0x10001u;
#pragma unroll
    for (uint32_t j = 0; j < W; ++j) R.m[j] = (R.m[j] & ~ins[j]) | (mv & ins[j]);
    if (LOG && s + 1u == next) log();
  }
  if (active) {
    const uint32_t tm = ns ? 0u : (uint32_t)(((uint64_t)t0 + steps) % L);
#pragma unroll
    for (uint32_t c = 0; c < NC; ++c) {
      const uint32_t xc = x + NS * c;
      if (xc < L)
        store_sites<NS>(M, xc, tm, L - xc, R.m + c * NS / 2, R.z + c * NS / 2, R.p + c * NS / 2);
    }
  }
}

// ---------------------------------------------------------------------------
// Lattices in tiles
// ---------------------------------------------------------------------------
// Positions of a lattice run over Lp = its sites rounded up to 8, so that a
// lane's chunks and the Philox calls stay in step across its end.  The (up to
// seven) positions L .. Lp - 1 hold no sites; streaming passes over them.

// The kh positions on each side of every boundary between two blocks' ranges
// at the launch's first step: strip s holds those from (the end of the range
// before it) - kh on, 2 kh per array.
__global__ void __launch_bounds__(64) k_strips(StepLaunch a, TileLaunch tl) {
  const StripDev sd = tl.strips[blockIdx.x];
  const SlotDev sl = a.slots[sd.slot];
  const Mem M = slot_mem(a.state, sl);
  const uint32_t L = M.L, Lp = (L + 7u) & ~7u, len = 2u * tl.kh;
  const uint32_t tm = a.p.no_stream ? 0u : (a.tslot[sd.slot] + a.t_off) % L;
  uint16_t *const out = tl.strip_data + (uint64_t)blockIdx.x * 3u * len;
  const Rsrc ors = __builtin_amdgcn_make_buffer_rsrc(out, 0, (int)(6u * len), kRsrcWord3);
  for (uint32_t i = 8u * threadIdx.x; i < len; i += 512u) {
    uint32_t x = ((sd.x + 7u) & ~7u) + Lp - tl.kh + i;
    x -= x >= Lp ? Lp : 0u;
    x -= x >= Lp ? Lp : 0u;
    uint32_t m[4], z[4], p[4];
    load_sites<8>(M, x, tm, true, 8u, m, z, p);
    vstore<8>(ors, 2u * i, 0u, m);
    vstore<8>(ors, 2u * i, 2u * len, z);
    vstore<8>(ors, 2u * i, 4u * len, p);
  }
}

// Block b takes the units [unit_first[b], unit_first[b + 1]) one after the
// other.  A unit is a whole lattice or a part [x0, x1) of one whose other
// parts other blocks hold; it is cut into tiles of up to 256 Q - 2 kh sites,
// consecutive ones to each wave.  In the in-place shifted layout a tile's
// write-back after K steps overwrites the step-t counts of up to K sites to
// either side of it, so each of those is read before anything is written:
// a wave's first tile, with its kh extra sites, and the sites around the end
// of its run of tiles (into its private area) before the block's barrier;
// the first 2 kh sites of every further tile when the tile before it was
// loaded (into the private area); and what lies within kh sites of another
// block's range from the strips, which k_strips wrote before the launch.
template <int Q, bool GAL, bool FIXED, bool LOG>
__global__ void __launch_bounds__(1024) k_tile(StepLaunch a, TileLaunch tl) {
  constexpr uint32_t S = 4u * Q, NS = Q == 1 ? 4 : 8, NC = S / NS;
  extern __shared__ uint4 lds[];
  const uint32_t lane = threadIdx.x & 63u, nw = blockDim.x >> 6;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t kh = tl.kh, slen = 2u * kh;
  const bool ns = a.p.no_stream != 0u, coll = a.p.C != 0;
  // the wave's private area: the positions around the end of its run, then two
  // carries (2 kh per array each)
  uint16_t *const priv =
      reinterpret_cast<uint16_t *>(a.overflow + (size_t)(blockIdx.x * nw + wave) * kOverflowPerWave);
  const Rsrc prs = __builtin_amdgcn_make_buffer_rsrc(priv, 0, (int)(16u * kOverflowPerWave), kRsrcWord3);
  auto carry_at = [&](uint32_t c) { return 6u * slen + c * 12u * kh; };
  uint64_t loaded = ~0ull;
  const uint32_t i0 = tl.unit_first[blockIdx.x], i1 = tl.unit_first[blockIdx.x + 1u];
  // the wave's records of the launch's logs (of one lattice) start empty
  for (uint32_t j = 0; LOG && j < tl.log.n; ++j)
    if (lane < kMom3Rec)
      tl.log.records[((uint64_t)j * tl.log.stride + blockIdx.x * nw + wave) * kMom3Rec + lane] = 0ull;
  for (uint32_t it = i0; it < i1; ++it) {
    const UnitDev un = tl.units[it];
    const uint32_t slot = __builtin_amdgcn_readfirstlane(un.slot);
    const uint32_t ux0 = __builtin_amdgcn_readfirstlane(un.x0);
    const uint32_t ux1 = __builtin_amdgcn_readfirstlane(un.x1);
    const bool split = __builtin_amdgcn_readfirstlane(un.split) != 0u;
    const uint32_t el = __builtin_amdgcn_readfirstlane(un.el);
    const uint32_t er = __builtin_amdgcn_readfirstlane(un.er);
    const SlotDev sl = a.slots[slot];
    const ImageDesc im = a.images[slot];
    const Mem M = slot_mem(a.state, sl);
    const uint32_t L = M.L, Lp = (L + 7u) & ~7u;
    const uint32_t t0 = __builtin_amdgcn_readfirstlane(a.tslot[slot] + a.t_off);
    const uint32_t tm = ns ? 0u : t0 % L;
    const uint32_t steps = __builtin_amdgcn_readfirstlane(tl.limit ? tl.limit[slot] : tl.steps);
    const uint32_t tmk = ns ? 0u : (uint32_t)(((uint64_t)t0 + steps) % L);
    // The unit's tiles, equal ones, dealt to the waves.  A SIMD issues for its
    // oldest wave first, so that with as many tiles for each of its four the
    // youngest ends long after the others, alone.  Wave 4 g + j gets them in
    // the ratio (64 + 3 s) : (64 + s) : (64 - s) : (64 - 3 s) of its g.  s is
    // the image's skew, smaller where more sites wait for a row (image_skew),
    // and smaller for few tiles, of which whole ones go to a wave: none up to
    // one per wave.  2^27 sites, Q = 6, us per step at s = 0: 203, 4: 188, 8:
    // 177, 10: 171, 12: 175, 16: 192.
    const uint32_t len = ux1 - ux0, tmax = 64u * S - 2u * kh;
    const uint32_t nt = max((len + tmax - 1u) / tmax, 4u);  // (T + 2 kh <= L, see kMinTiled)
    const uint32_t T = ((len + nt - 1u) / nt + 7u) / 8u * 8u;
    const uint32_t ntile = (len + T - 1u) / T;
    const uint32_t group = wave >> 2, groups = nw >> 2;
    const uint32_t skew =
        __builtin_amdgcn_readfirstlane(ntile > nw ? im.skew * (ntile - nw) / ntile : 0u);
    auto share = [&](uint32_t g) {  // tiles of each of the group's waves, rounded down
      return ntile * (64u + (groups - 1u) * skew - 2u * skew * g) / (256u * groups);
    };
    uint32_t ta = (wave & 3u) * share(group), left = ntile;
    for (uint32_t g = 0; g < groups; ++g) {
      left -= 4u * share(g);
      ta += g < group ? 4u * share(g) : 0u;
    }
    // (fewer than 4 groups are left: one each for the oldest)
    const uint32_t tb0 = ta + share(group);
    ta += min(wave, left);
    const uint32_t tb = tb0 + min(wave, left) + (wave < left ? 1u : 0u);
    const uint32_t X0 = ux0 + ta * T, end = min(ux1, ux0 + tb * T);  // the wave's run
    const uint32_t endp = (end + 7u) & ~7u, ux1p = (ux1 + 7u) & ~7u;
    const Rsrc lrs = __builtin_amdgcn_make_buffer_rsrc(
        tl.strip_data + (uint64_t)(split ? el : 0u) * 3u * slen, 0, (int)(6u * slen), kRsrcWord3);
    const Rsrc rrs = __builtin_amdgcn_make_buffer_rsrc(
        tl.strip_data + (uint64_t)(split ? er : 0u) * 3u * slen, 0, (int)(6u * slen), kRsrcWord3);
    auto load_area = [&](Rsrc rs, uint32_t at, uint32_t ah, uint32_t *m, uint32_t *z, uint32_t *p) {
      vload<NS>(rs, at, 0u, m);
      vload<NS>(rs, at + ah, 0u, z);
      vload<NS>(rs, at + 2u * ah, 0u, p);
    };
    // NS positions from y on (-kh <= y < Lp + kh) at the launch's first step,
    // from the state as the launch found it
    auto load_first = [&](int32_t y, uint32_t *m, uint32_t *z, uint32_t *p) {
      if (split && y < (int32_t)(ux0 + kh)) {
        load_area(lrs, 2u * ((uint32_t)y + kh - ux0), 2u * slen, m, z, p);
      } else if (split && y >= (int32_t)(ux1p - kh)) {
        load_area(rrs, 2u * ((uint32_t)y - (ux1p - kh)), 2u * slen, m, z, p);
      } else {
        uint32_t x = y < 0 ? (uint32_t)(y + (int32_t)Lp) : (uint32_t)y;
        x -= x >= Lp ? Lp : 0u;
        load_sites<NS>(M, x, tm, true, NS, m, z, p);
      }
    };
    __syncthreads();  // the image before is no longer in use
    const Env E{lds + a.lds_bytes / 16u + wave * (kWaveLdsBytes / 16u),
                make_uint2((uint32_t)a.p.seed, (uint32_t)(a.p.seed >> 32)), image_view(im), (L + 7u) & ~7u, sl.rid, lane};
    const bool active = ta < tb;
    Sites<Q> R;
    uint32_t cpar = 0;
    // the tile at xt: n sites, positions kh .. kh + n - 1 of the wave.  The
    // positions after its extra sites repeat it from the start (and the
    // wave's ends meet): their values are never used, but being counts like
    // the others they miss the image no more often, as empty sites would.
    auto load_tile = [&](uint32_t xt, uint32_t n, bool first) {
      const uint32_t es = ((n + 7u) & ~7u) + 2u * kh;
#pragma unroll
      for (uint32_t c = 0; c < NC; ++c) {
        uint32_t *const m = R.m + c * NS / 2, *const z = R.z + c * NS / 2, *const p = R.p + c * NS / 2;
        const uint32_t i0_ = lane * S + c * NS, i = i0_ % es;
        const int32_t y = (int32_t)(xt + i) - (int32_t)kh;
        if (first) {
          load_first(y, m, z, p);
        } else if (i < 2u * kh) {
          load_area(prs, carry_at(cpar ^ 1u) + 2u * i, 4u * kh, m, z, p);
        } else if (y >= (int32_t)(endp - kh)) {
          load_area(prs, 2u * ((uint32_t)y - (endp - kh)), 2u * slen, m, z, p);
        } else {
          load_sites<NS>(M, (uint32_t)y, tm, true, NS, m, z, p);
        }
        if (xt + n < end && i0_ >= n && i0_ < n + 2u * kh) {  // the next tile's first 2 kh sites
          const uint32_t at = carry_at(cpar) + 2u * (i - n);
          vstore<NS>(prs, at, 0u, m);
          vstore<NS>(prs, at + 4u * kh, 0u, z);
          vstore<NS>(prs, at + 8u * kh, 0u, p);
        }
      }
      cpar ^= 1u;
    };
    if (active) load_tile(X0, min(T, end - X0), true);
    if (im.off != loaded) copy_image(lds, a.image_pool, im);
    loaded = im.off;
    if (active) {
      if (tb - ta > 1u) {
        for (uint32_t i = 8u * lane; i < slen; i += 512u) {
#pragma unroll
          for (uint32_t h = 0; h < 8u; h += NS) {
            uint32_t m[NS / 2], z[NS / 2], p[NS / 2];
            load_first((int32_t)(endp + i + h) - (int32_t)kh, m, z, p);
            vstore<NS>(prs, 2u * (i + h), 0u, m);
            vstore<NS>(prs, 2u * (i + h) + 2u * slen, 0u, z);
            vstore<NS>(prs, 2u * (i + h) + 4u * slen, 0u, p);
          }
        }
      }
    }
    __syncthreads();  // everything of the launch's first step is read; the image is in place
    if (!active) continue;
    for (uint32_t k = ta; k < tb; ++k) {
      const uint32_t xt = ux0 + k * T, n = min(T, end - xt);
      if (k != ta) {
        __threadfence_block();  // the private area's stores
        load_tile(xt, n, false);
      }
      Span Sp;
      Sp.end = 64u * S;
      Sp.own_lo = kh;
      Sp.own_hi = kh + n;
      Sp.slow = false;
      const uint32_t pos = lane * S;
      const uint32_t xw = xt >= kh ? xt - kh : xt + Lp - kh;
      // where the lattice's site 0 comes after its last one in this tile,
      // with positions without sites between them
      const uint32_t pad = Lp - L, p0 = xt < kh ? kh - xt : Lp + kh - xt;
      const bool seam = pad != 0u && !ns && p0 < 64u * S && p0 > pad;
      uint32_t next = LOG ? tl.log.first : 0u, logs = 0;
      for (uint32_t s = 0; s < steps; ++s) {
        collide<Q, GAL, FIXED>(R, E, xw, Sp, t0 + s, coll);
        if (!ns) {
        uint32_t up = 0, down = 0;
        if (seam) {
          up = site_of<Q>(R.p, p0 - 1u - pad);
          down = site_of<Q>(R.m, p0);
        }
        stream<Q, true>(R, 0u, 0u);
        if (seam) {
          set_site<Q>(R.p, p0, lane, up);
          set_site<Q>(R.m, p0 - 1u - pad, lane, down);
        }
        }
        if (LOG && s + 1u == next) {
          const RegLog *lg = log_args<TileLaunch>();
          log_sites<Q>(R, xw, Lp, L, kh, kh + min(n, L - xt), lg, lg->tw,
                       lg->records + ((uint64_t)logs * lg->stride + blockIdx.x * nw + wave) * kMom3Rec,
                       false);
          ++logs;
          next = logs < tl.log.n ? next + tl.log.every : 0u;
        }
      }
#pragma unroll
      for (uint32_t c = 0; c < NC; ++c) {
        const uint32_t i = pos + c * NS;
        if (i >= kh && i < kh + n)
          store_sites<NS>(M, xt + i - kh, tmk, kh + n - i, R.m + c * NS / 2, R.z + c * NS / 2,
                          R.p + c * NS / 2);
      }
    }
  }
}
}  // namespace

template <typename K>
static hipError_t allow_lds(K kernel, uint32_t lds) {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

uint32_t reg_lds_bytes(uint32_t image_bytes, uint32_t waves) {
  return (image_bytes + 15u) / 16u * 16u + waves * kWaveLdsBytes + kRingExchangeBytes;
}

hipError_t reg_setup(uint32_t image_bytes) {
  const uint32_t lds = reg_lds_bytes(image_bytes, 16);
  hipError_t e = hipSuccess;
#define MCLG_ALLOW(...)                                     \
  if (!e) e = allow_lds(k_ring<__VA_ARGS__>, lds);          \
  if (!e) e = allow_lds(k_tile<__VA_ARGS__>, lds);
  MCLG_ALLOW(1, false, true, false) MCLG_ALLOW(2, false, true, false)
  MCLG_ALLOW(4, false, true, false) MCLG_ALLOW(6, false, true, false)
  MCLG_ALLOW(1, true, true, false) MCLG_ALLOW(2, true, true, false)
  MCLG_ALLOW(2, false, false, false) MCLG_ALLOW(2, true, false, false)
  MCLG_ALLOW(1, false, true, true) MCLG_ALLOW(2, false, true, true)
  MCLG_ALLOW(4, false, true, true)
#undef MCLG_ALLOW
  return e;
}

// The instantiations: images of fixed records for every Q (the Galilean
// acceptance, whose literal loop needs the registers, for Q <= 2), the others
// (C = infinity or C > 20) for Q = 2; logs with the constant acceptance and
// fixed records for Q <= 4 (a log's sums take the registers of two more).
bool reg_has(uint32_t Q, bool galilean, bool fixed, bool logs) {
  if (Q != 1 && Q != 2 && Q != 4 && Q != 6) return false;
  if (logs) return !galilean && fixed && Q <= 4;
  return fixed ? !galilean || Q <= 2 : Q == 2;
}
#define MCLG_REG_LAUNCH(KERNEL, GRID, ARGS)                                              \
  switch (Q + (a.p.galilean ? 8u : 0u) + (images_fixed(a.p.C) ? 0u : 16u) + (ARGS.log.n ? 32u : 0u)) { \
    case 1: KERNEL<1, false, true, false><<<GRID, block, lds, s>>>(a, ARGS); break;      \
    case 2: KERNEL<2, false, true, false><<<GRID, block, lds, s>>>(a, ARGS); break;      \
    case 4: KERNEL<4, false, true, false><<<GRID, block, lds, s>>>(a, ARGS); break;      \
    case 6: KERNEL<6, false, true, false><<<GRID, block, lds, s>>>(a, ARGS); break;      \
    case 9: KERNEL<1, true, true, false><<<GRID, block, lds, s>>>(a, ARGS); break;       \
    case 10: KERNEL<2, true, true, false><<<GRID, block, lds, s>>>(a, ARGS); break;      \
    case 18: KERNEL<2, false, false, false><<<GRID, block, lds, s>>>(a, ARGS); break;    \
    case 26: KERNEL<2, true, false, false><<<GRID, block, lds, s>>>(a, ARGS); break;     \
    case 33: KERNEL<1, false, true, true><<<GRID, block, lds, s>>>(a, ARGS); break;      \
    case 34: KERNEL<2, false, true, true><<<GRID, block, lds, s>>>(a, ARGS); break;      \
    case 36: KERNEL<4, false, true, true><<<GRID, block, lds, s>>>(a, ARGS); break;      \
    default: return hipErrorInvalidValue;                                                \
  }

static bool log_ok(const RegLog &lg, uint32_t steps, uint32_t stride) {
  return lg.n == 0 || (lg.first >= 1 && lg.every >= 1 && lg.n_modes <= 8 && lg.records && lg.out &&
                       (lg.tw || lg.n_modes == 0) && lg.stride >= stride &&
                       lg.first + (uint64_t)(lg.n - 1u) * lg.every <= steps);
}

hipError_t launch_ring(hipStream_t s, const StepLaunch &a, const RingLaunch &rl, uint32_t Q,
                       uint32_t waves) {
  if (rl.n == 0 || rl.steps == 0) return hipSuccess;
  if (waves < 1 || waves > 16 || rl.team > waves || !log_ok(rl.log, rl.steps, rl.team ? 1u : waves) ||
      (rl.log.n && rl.limit))
    return hipErrorInvalidValue;
  const dim3 grid(rl.team ? (rl.n + rl.team - 1u) / rl.team : rl.n), block(64u * waves);
  const uint32_t lds = reg_lds_bytes(a.lds_bytes, waves);
  MCLG_REG_LAUNCH(k_ring, grid, rl)
  if (rl.log.n) k_log_final<<<rl.log.n * rl.n, 256, 0, s>>>(a, rl.log, rl.order, rl.n, a.t_off);
  return hipGetLastError();
}

hipError_t launch_tiles(hipStream_t s, const StepLaunch &a, const TileLaunch &tl, uint32_t Q,
                        uint32_t waves, uint32_t grid, const uint32_t *order) {
  if (tl.steps == 0) return hipSuccess;
  // the tiles' own sites, the private areas and their number; logs of one
  // lattice only
  if (waves < 4 || waves > 16 || waves % 4u || tl.kh % 8u != 0u || tl.steps > tl.kh || 2u * tl.kh >= 256u * Q ||
      36u * tl.kh > 16u * kOverflowPerWave || grid * waves > kOverflowWaves ||
      !log_ok(tl.log, tl.steps, grid * waves) || (tl.log.n && (a.n_slots != 1u || tl.limit)))
    return hipErrorInvalidValue;
  if (tl.n_strips) {
    k_strips<<<tl.n_strips, 64, 0, s>>>(a, tl);
    hipError_t e = hipGetLastError();
    if (e) return e;
  }
  const dim3 g(grid), block(64u * waves);
  const uint32_t lds = reg_lds_bytes(a.lds_bytes, waves);
  MCLG_REG_LAUNCH(k_tile, g, tl)
  if (tl.log.n) k_log_final<<<tl.log.n, 1024, 0, s>>>(a, tl.log, order, 1u, a.t_off);
  return hipGetLastError();
}

}  // namespace mclg
