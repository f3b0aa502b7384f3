// HIP kernels of the MCLG library for gfx950 (MI355X).
//
// The hot kernel fuses streaming and the Monte Carlo collision of the D1Q3
// integer lattice gas (Sec. "The Monte Carlo Lattice Gas algorithm" and
// "A D1Q3 implementation"): per site it loads n_-1, n_0, n_+1 (uint16) from
// the in-place shifted layout, draws the post-collision rest count from the
// exact C-sub-collision law with one Philox4x32-10 word, restores n_-1 and
// n_+1 from the conserved N and J, and stores the three counts back to the
// same three physical locations -- streaming is the shift of the layout.
// Algorithmic traffic: 6 B read + 6 B written per site update; there is no
// dense contraction, so no MFMA.
#include "collide.h"
#include "device.h"
#include "rng.h"


#include <algorithm>

namespace mclg {
namespace {

// Per-wave queue of draws the LDS image could not decide (or sites with
// N > n_max); drained by all lanes at once.
constexpr uint32_t kOverflow = kOverflowPerWave;

// Where a slot's three arrays are and how they are shifted at step t.
struct SlotView {
  uint32_t lo, hi;  // address of the slot's n_-1 array; n_0 and n_+1 follow
  uint32_t ab;      // bytes per array
  uint32_t L, tm, t, rid;
  // the buffer resource, rebuilt at each use from wave-uniform scalars
  __device__ __forceinline__ Rsrc rs() const {
    return __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<void *>(((uint64_t)hi << 32) | lo), 0, (int)(3u * ab), kRsrcWord3);
  }
};

// The wave's queue of undecided draws: a virtual array of kQueue entries in
// LDS followed by kOverflow entries in global memory, filled to F
// (wave-uniform).  An entry is (x, a | b << 16, c, r) with the site's
// pre-collision counts; the chunk stores whatever its lane computed for such
// a site, and the drain overwrites it with the exact outcome.  When the
// chunk's draws are resolved before its store (kDrainPatch), the first word
// is instead the site's position in the chunk, 8 lane + K.
static_assert(kDrainAt + 512 <= kQueue + kOverflow, "a chunk's draws must fit the queue");

// Site K of every lane in mk, whose draw was not decided (and, in a chunk that
// passes the end of the lattice, that exists) goes to the queue, in lane
// order.  wa, wb, wc are the words holding the site's pre-collision counts;
// `slow` is wave-uniform.
template <int K, bool PATCH>
__device__ __forceinline__ void push_site(uint4 *queue, Rsrc over, uint32_t &F, uint64_t mk,
                                          bool slow, uint32_t x8, uint32_t L, uint32_t wa,
                                          uint32_t wb, uint32_t wc, uint32_t r, uint32_t xs) {
  if (mk == 0) return;
  if (slow) mk &= lanes_gt(L, x8 + K);
  const uint32_t n = (uint32_t)__popcll(mk);
  if (__builtin_amdgcn_inverse_ballot_w64(mk)) {
    const uint32_t pos = F + lanes_below(mk);
    const uint32_t ab = (K & 1) ? __builtin_amdgcn_perm(wb, wa, 0x07060302u)
                                : __builtin_amdgcn_perm(wb, wa, 0x05040100u);
    const uint32_t c = (K & 1) ? wc >> 16 : wc & 0xffffu;
    uint32_t w0 = x8 + K;
    if constexpr (PATCH) {
      // the position in the chunk (xs: its first site), computed here rather
      // than hoisted out of the chunk loop as a per-lane constant
      w0 -= xs;
      asm volatile("" : "+v"(w0));
    }
    if (pos < kQueue) {
      queue[pos] = make_uint4(w0, ab, c, r);
    } else {
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      const u32x4 e = {w0, ab, c, r};
      __builtin_amdgcn_raw_buffer_store_b128(e, over, (int)(16u * (pos - kQueue)), 0, 0);
    }
  }
  F += n;
}

// All eight sites of the lane: directory reads of all eight first, the
// Philox draws while they are in flight, then record reads and decisions;
// the undecided draws are queued with the pre-collision counts before the
// update.
template <bool PATCH, bool FIXED>
__device__ __forceinline__ void decide_eight(uint4 &w0, uint4 &w1, uint2 key,
                                             uint32_t (&va)[4], uint32_t (&vb)[4],
                                             uint32_t (&vc)[4], const LdsView &lv, uint4 *queue,
                                             Rsrc over, uint32_t &F, bool slow, uint32_t x8,
                                             uint32_t L, uint32_t xs) {
  SiteLook s0, s1, s2, s3, s4, s5, s6, s7;
  uint32_t r0, r1, r2, r3, r4, r5, r6, r7;  // each site's first record
  u16x2 b01, b23, b45, b67;                  // clamped b - b_lo of each pair
  site_dir_pair<0>(r0, r1, b01, va, vb, vc, lv);
  site_dir_pair<1>(r2, r3, b23, va, vb, vc, lv);
  site_dir_pair<2>(r4, r5, b45, va, vb, vc, lv);
  site_dir_pair<3>(r6, r7, b67, va, vb, vc, lv);
  philox10_x2(w0, w1, key);
  rec_pair(s0, s1, r0, r1, b01);
  rec_pair(s2, s3, r2, r3, b23);
  rec_pair(s4, s5, r4, r5, b45);
  rec_pair(s6, s7, r6, r7, b67);
  uint64_t h0, h1, h2, h3, h4, h5, h6, h7;  // lanes whose site is undecided
  const uint32_t d01 = finish_pair<FIXED>(s0, s1, w0.x, w0.y, lv, h0, h1);
  const uint32_t d23 = finish_pair<FIXED>(s2, s3, w0.z, w0.w, lv, h2, h3);
  const uint32_t d45 = finish_pair<FIXED>(s4, s5, w1.x, w1.y, lv, h4, h5);
  const uint32_t d67 = finish_pair<FIXED>(s6, s7, w1.z, w1.w, lv, h6, h7);
  uint32_t na[4] = {va[0], va[1], va[2], va[3]}, nb[4] = {vb[0], vb[1], vb[2], vb[3]},
           nc[4] = {vc[0], vc[1], vc[2], vc[3]};
  apply_pair(na[0], nb[0], nc[0], d01);
  apply_pair(na[1], nb[1], nc[1], d23);
  apply_pair(na[2], nb[2], nc[2], d45);
  apply_pair(na[3], nb[3], nc[3], d67);
#define MCLG_PUSH(K, H, R)                                                                \
  push_site<K, PATCH>(queue, over, F, H, slow, x8, L, va[K >> 1], vb[K >> 1], vc[K >> 1], R, \
                      xs)
  MCLG_PUSH(0, h0, w0.x); MCLG_PUSH(1, h1, w0.y); MCLG_PUSH(2, h2, w0.z); MCLG_PUSH(3, h3, w0.w);
  MCLG_PUSH(4, h4, w1.x); MCLG_PUSH(5, h5, w1.y); MCLG_PUSH(6, h6, w1.z); MCLG_PUSH(7, h7, w1.w);
#undef MCLG_PUSH
  for (int j = 0; j < 4; ++j) {
    va[j] = na[j];
    vb[j] = nb[j];
    vc[j] = nc[j];
  }
}

// Without collisions only a site whose N does not fit 16 bits is queued
// (the drain flags it and keeps its counts).
template <bool PATCH>
__device__ __forceinline__ void queue_saturated(const uint32_t (&va)[4], const uint32_t (&vb)[4],
                                                const uint32_t (&vc)[4], uint4 *queue,
                                                Rsrc over, uint32_t &F, bool slow,
                                                uint32_t x8, uint32_t L, uint32_t xs) {
#define MCLG_SAT(J)                                                                              \
  {                                                                                              \
    const uint32_t N2 = __builtin_bit_cast(                                                      \
        uint32_t, __builtin_elementwise_add_sat(                                                 \
                      __builtin_elementwise_add_sat(__builtin_bit_cast(u16x2, va[J]),            \
                                                    __builtin_bit_cast(u16x2, vb[J])),           \
                      __builtin_bit_cast(u16x2, vc[J])));                                        \
    push_site<2 * J, PATCH>(queue, over, F, lanes_eq(N2 & 0xffffu, 0xffffu), slow, x8, L, va[J],      \
                            vb[J], vc[J], 0u, xs);                                               \
    push_site<2 * J + 1, PATCH>(queue, over, F, lanes_eq(N2 >> 16, 0xffffu), slow, x8, L, va[J],      \
                                vb[J], vc[J], 0u, xs);                                           \
  }
  MCLG_SAT(0) MCLG_SAT(1) MCLG_SAT(2) MCLG_SAT(3)
#undef MCLG_SAT
}

// Resolve every queued draw of the wave (all lanes in parallel) and store
// the site's three final counts.  The wave first waits until all of its
// earlier memory operations have completed -- among them the stores that
// wrote the pre-collision counts of these sites -- so the final counts land
// after them.
template <bool GAL>
__device__ __forceinline__ void drain_queue(const uint4 *queue, const uint4 *over, uint32_t F,
                                            uint32_t lane, const SlotView &v,
                                            const StepParams &p, const TableDev &tab,
                                            uint32_t *err) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_waitcnt(0);  // vmcnt = expcnt = lgkmcnt = 0
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  for (uint32_t i = lane; i < F; i += 64u) {
    const uint4 e = i < kQueue ? queue[i] : over[i - kQueue];
    const uint32_t x = e.x, ea = e.y & 0xffffu, eb = e.y >> 16, ec = e.z;
    const uint32_t bn =
        resolve_queued<GAL>(e, p, tab, v.t, v.rid, err);
    const int32_t N = (int32_t)(ea + eb + ec), J = (int32_t)ec - (int32_t)ea;
    uint32_t pm = x + v.tm;
    pm -= (pm >= v.L) ? v.L : 0u;
    const uint32_t pp = x >= v.tm ? x - v.tm : x + v.L - v.tm;
    bstore2(v.rs(), 2u * pm, 0u, (uint32_t)((N - (int32_t)bn - J) >> 1));
    bstore2(v.rs(), 2u * x, v.ab, bn);
    bstore2(v.rs(), 2u * pp, 2u * v.ab, (uint32_t)((N - (int32_t)bn + J) >> 1));
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

// The move decide_eight applied to one undecided site (a, b, c; draw r):
// the same directory and record reads from the LDS image, one site in
// 32-bit arithmetic with the 16-bit wrap-around of the packed form.
template <bool FIXED>
__device__ __forceinline__ uint32_t image_move(uint32_t a, uint32_t b, uint32_t c, uint32_t r,
                                               const LdsView &lv) {
  const uint32_t lo = min(min(a, c), lv.da2 & 0xffffu), hi = min(max(a, c), lv.dc2 & 0xffffu);
  const uint32_t row = lds_u32((lo * (lv.w4 & 0xffffu) + 4u * hi) & 0xffffu);
  const uint32_t bi = min((b - (lv.blo2 & 0xffffu)) & 0xffffu, lv.nb2 & 0xffffu);
  SiteLook sl;
  sl.q = lds_u4(row + 16u * bi);
  uint64_t miss;
  return site_finish<FIXED>(sl, r, lv, miss) & 0xffffu;
}

// Resolve the draws queued by the current chunk before its store
// (kDrainPatch): each lane takes one entry at a time, finds the exact outcome
// and writes the correction of the move the site's lane applied (found again
// from the image), as a 16-bit patch at the site's position; the LDS queue's
// 1 KB holds the chunk's 512 patches once its entries have been read.  Every
// lane then adds its eight patches to its counts (zero for decided sites), so
// the chunk's vector stores write the final counts.
template <bool GAL, bool FIXED>
__device__ __forceinline__ void patch_chunk(uint4 *queue, const uint4 *over, uint32_t F,
                                            uint32_t lane, uint32_t xs, const SlotView &v,
                                            const LdsView &lv, const StepParams &p,
                                            const TableDev &tab, uint32_t *err, uint32_t (&m)[4],
                                            uint32_t (&z)[4], uint32_t (&c)[4]) {
  if (F > kQueue) {
    // entries past the LDS queue were written to global memory by other
    // lanes: wait for those stores before reading them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  }
  const uint4 e0 = lane < F ? queue[lane] : make_uint4(0u, 0u, 0u, 0u);
  // each lane clears its own 16 bytes (its eight sites' patches) after
  // reading the entry stored there
  queue[lane] = make_uint4(0u, 0u, 0u, 0u);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  uint16_t *const patch = reinterpret_cast<uint16_t *>(queue);
  for (uint32_t i = lane; i < F; i += 64u) {
    uint4 e = i < kQueue ? e0 : over[i - kQueue];
    const uint32_t pos = e.x, b = e.y >> 16;
    // C = 0 queues only overflowing sites and applies no move
    const uint32_t dw = p.C != 0 ? image_move<FIXED>(e.y & 0xffffu, b, e.z, e.w, lv) : 0u;
    e.x = xs + pos;
    const uint32_t bn = resolve_queued<GAL>(e, p, tab, v.t, v.rid, err);
    const uint32_t d = (uint32_t)(((int32_t)b - (int32_t)bn) >> 1);
    patch[pos] = (uint16_t)(d - dw);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const uint4 pv = queue[lane];
  apply_pair(m[0], z[0], c[0], pv.x);
  apply_pair(m[1], z[1], c[1], pv.y);
  apply_pair(m[2], z[2], c[2], pv.z);
  apply_pair(m[3], z[3], c[3], pv.w);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Streaming over a wave's run of consecutive chunks
// ---------------------------------------------------------------------------
// Where chunk xs .. xs + 511 of a slot lies at step t: the three physical
// windows (n_-1 at (x + t) mod L, n_0 at x, n_+1 at (x - t) mod L) and
// whether none of them wraps around the end of the lattice (fast path).
struct Win {
  uint32_t xs, sm, sp;
  uint32_t fast;  // 0 or 1
};
__device__ __forceinline__ Win locate(uint32_t xs, const SlotView &v) {
  Win w;
  w.xs = xs;
  w.sm = xs + v.tm;
  w.sm -= (w.sm >= v.L) ? v.L : 0u;
  w.sp = xs >= v.tm ? xs - v.tm : xs + v.L - v.tm;
  w.fast = (uint32_t)((xs + 512u <= v.L) & (w.sm + 512u <= v.L) & (w.sp + 512u <= v.L));
  return w;
}
// A fast chunk's three windows, one 16-byte access per lane each: lane i
// owns elements s + 8 i .. s + 8 i + 7 of every window.  The n_+-1 windows
// start at any element (2-byte alignment); the hardware serves unaligned
// vector accesses, and neighbouring lanes, chunks and waves touch disjoint
// bytes, so each lane reads and writes exactly its own eight elements.
struct Raw {
  uint32_t m[4], z[4], p[4];
};
template <int CP>
__device__ __forceinline__ void issue_raw(const Win &w, const SlotView &v, uint32_t lane,
                                          Raw &r) {
  const uint32_t vo = 16u * lane;
  bload4<CP>(v.rs(), vo, 2u * w.sm, r.m);
  bload4<CP>(v.rs(), vo, v.ab + 2u * w.xs, r.z);
  bload4<CP>(v.rs(), vo, 2u * v.ab + 2u * w.sp, r.p);
}
// The chunk's three windows as eight consecutive sites per lane, in place in
// `r`: a fast chunk's vectors are there already; a chunk whose windows wrap
// around the end of the lattice (or pass it) is read element by element.
// Sites past the end read as empty (N = 0) and are never stored.
__device__ __forceinline__ void chunk_fill(const Win &w, Raw &r, const SlotView &v,
                                           uint32_t lane) {
  if (!w.fast) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t x = w.xs + 8u * lane + e;
      uint32_t ea = 0, eb = 0, ec = 0;
      if (x < v.L) {
        uint32_t pm = x + v.tm;
        pm -= (pm >= v.L) ? v.L : 0u;
        const uint32_t pp = x >= v.tm ? x - v.tm : x + v.L - v.tm;
        ea = bload2(v.rs(), 2u * pm, 0u);
        eb = bload2(v.rs(), 2u * x, v.ab);
        ec = bload2(v.rs(), 2u * pp, 2u * v.ab);
      }
      set16(r.m, e, ea); set16(r.z, e, eb); set16(r.p, e, ec);
    }
  }
  // complete here, so that no load of this chunk is still counted when the
  // next chunk's loads are issued
  for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(r.m[j]), "+v"(r.z[j]), "+v"(r.p[j]));
}

// The block's next chunk index (an LDS counter), wave-uniform.
__device__ __forceinline__ uint32_t grab_chunk(uint32_t *ctr, uint32_t lane) {
  uint32_t v = 0;
  if (lane == 0) v = atomicAdd(ctr, 1u);
  return __builtin_amdgcn_readfirstlane(v);
}

// Fused stream + collide.  Persistent blocks: block i takes a contiguous
// range of chunks; the slot's collision image is loaded into LDS for each
// run of one slot's chunks (a segment), whose chunks the block's waves then
// claim one at a time.  Each wave keeps one chunk of lookahead: the next
// chunk's vectors are requested before the current one is decided.  Each
// lane owns 8 consecutive sites of a chunk (two Philox calls).  Every
// physical element belongs to exactly one site per step, so the in-place
// update has no races.  Undecided draws wait in the wave's queue, which is
// drained between chunks once it nears capacity, and at the end of the
// slot's segment.
// FIXED: the images hold fixed records (see LdsImage), whose decision needs no
// masks that depend on the image: 2^24 sites of density 50, 37.8 us per step
// and 38.4 with them, 2^22 14.6 and 15.3.
template <int MAXT, bool GAL, int MODE, bool FIXED>
__global__ void __launch_bounds__(MAXT) k_step(StepLaunch a) {
  constexpr bool PATCH = MODE == kDrainPatch;
  // patched drains are the policy for states larger than the caches: their
  // chunk vectors are read and written as streaming (non-temporal) accesses
  constexpr int CP = PATCH ? kStreamingPolicy : 0;
  extern __shared__ uint4 lds[];
  const StepParams &p = a.p;
  const uint2 key = make_uint2((uint32_t)p.seed, (uint32_t)(p.seed >> 32));
  const uint32_t lane = threadIdx.x & 63u, nwaves = blockDim.x >> 6;
  // wave-uniform, which the compiler cannot infer from threadIdx.x
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint4 *const queue = lds + a.lds_bytes / 16u + wave * (kWaveLdsBytes / 16u);
  uint4 *const over = a.overflow + (size_t)(blockIdx.x * nwaves + wave) * kOverflow;
  const Rsrc ovr = __builtin_amdgcn_make_buffer_rsrc(over, 0, (int)(16u * kOverflow), kRsrcWord3);
  uint32_t F = 0;  // queue fill (wave-uniform), all draws of slot `cur`
  // Waves are spread over the four SIMDs in order, and the hardware issues
  // a SIMD's younger waves after its older ones, so a chunk held by a young
  // wave at the end of a segment finishes last: the youngest wave of each
  // SIMD stops claiming once at most nwaves chunks are left, the next
  // youngest once at most nwaves / 2 are.  The oldest wave of each SIMD
  // always claims, so every chunk is taken.
  const bool youngest = nwaves >= 8u && wave + 4u >= nwaves;
  const bool second = nwaves >= 12u && wave + 8u >= nwaves && !youngest;
  // after the image and the queues: the block's next unclaimed chunk of the
  // segment, and the last-block flag (so that the image starts at LDS 0)
  uint32_t *const ctl =
      reinterpret_cast<uint32_t *>(lds + a.lds_bytes / 16u + nwaves * (kWaveLdsBytes / 16u));
  uint32_t &next_chunk = ctl[0];
  const uint32_t per = (a.n_tiles + gridDim.x - 1) / gridDim.x;
  const uint32_t cb = blockIdx.x * per;
  const uint32_t ce = min(a.n_tiles, cb + per);
  uint32_t cur = 0xFFFFFFFFu;
  uint64_t img_off = ~0ull;  // pool offset of the image in LDS
  SlotView sv;
  sv.lo = sv.hi = 0;
  sv.ab = 0;
  sv.L = 1; sv.tm = sv.t = sv.rid = 0;
  LdsView lv;
  lv = image_view(ImageDesc{});

  for (uint32_t i = cb;;) {
    TileDev t0;
    t0.slot = cur;
    if (i < ce) {
      if (a.single) {
        t0.slot = a.slot_first;
        t0.x0 = i * 512u;
        t0.next = a.n_tiles;
      } else {
        t0 = a.tiles[i];
      }
    }
    if (!PATCH && F && (i >= ce || t0.slot != cur)) {  // queued draws belong to slot `cur`
      drain_queue<GAL>(queue, over, F, lane, sv, p, a.tab, a.err);
      F = 0;
    }
    if (i >= ce) break;
    t0.x0 = __builtin_amdgcn_readfirstlane(t0.x0);
    const uint32_t se = __builtin_amdgcn_readfirstlane(min(ce, t0.next));
    // Each wave's first chunk of the segment is fixed, so that its loads are
    // in flight while the image is copied; the rest go to the block's waves
    // one at a time from a shared counter, so that waves issued less often
    // (the hardware favours older waves) take fewer chunks and all finish
    // together.
    const bool first = cur == 0xFFFFFFFFu;
    cur = t0.slot;
    const ImageDesc im = a.single ? a.im1 : a.images[cur];
    // replicas that share an image keep it in LDS from segment to segment
    const bool new_image = first || im.off != img_off;
    img_off = im.off;
    const SlotDev sl = a.single ? a.sl1 : a.slots[cur];
    const uint32_t tn = a.tslot[cur] + a.t_off;
    if (!first) __syncthreads();  // previous image and chunk counter no longer in use
    // (wave-uniform values kept in scalar registers)
    sv.t = __builtin_amdgcn_readfirstlane(tn);
    sv.L = __builtin_amdgcn_readfirstlane(sl.L);
    sv.tm = p.no_stream ? 0u : sv.t % sv.L;
    sv.rid = __builtin_amdgcn_readfirstlane(sl.rid);
    const uint64_t base = reinterpret_cast<uint64_t>(a.state + sl.off);
    sv.lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
    sv.hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    sv.ab = __builtin_amdgcn_readfirstlane(2u * sl.stride);
    uint32_t k = min(i + wave, se);
    if (threadIdx.x == 0) next_chunk = i + nwaves;
    Win cw = locate(t0.x0 + (k - i) * 512u, sv);
    Raw cr;
    if (k < se && cw.fast) issue_raw<CP>(cw, sv, lane, cr);
    if (new_image) {
      // ten independent 16-byte loads per thread per round (a 1024-thread
      // block moves 160 KiB in one round), then the stores (indices clamped
      // into the image; the stores past its end are skipped)
      const uint4 *src = reinterpret_cast<const uint4 *>(a.image_pool + im.off);
      const uint32_t n16 = im.bytes / 16u, bd = blockDim.x, last = n16 - 1u;
      for (uint32_t b0 = threadIdx.x; b0 < n16; b0 += 10u * bd) {
        uint4 v[10];
#pragma unroll
        for (uint32_t j = 0; j < 10; ++j) v[j] = src[min(b0 + j * bd, last)];
        // all ten loads are issued before the first store waits for its data
        // (otherwise the compiler moves each load into its store's branch)
#pragma unroll
        for (uint32_t j = 0; j < 10; ++j)
          asm volatile("" : "+v"(v[j].x), "+v"(v[j].y), "+v"(v[j].z), "+v"(v[j].w));
        lds[b0] = v[0];
#pragma unroll
        for (uint32_t j = 1; j < 10; ++j)
          if (b0 + j * bd < n16) lds[b0 + j * bd] = v[j];
      }
      lv = image_view(im);
    }
    __syncthreads();  // the image and the counter are in place
    const uint32_t L = sv.L, tm = sv.tm, t = sv.t;  // of the segment's slot
    const Rsrc rs = sv.rs();
    const uint32_t ab = sv.ab;
    // One chunk: the next chunk's loads go out first (into the other
    // register set; its bytes are disjoint from this chunk's), then this
    // chunk is decided and stored, then the next chunk's vectors are taken.
    // The loop alternates the two register sets, so nothing is copied.
    auto one = [&](Raw &cur, Raw &nxt) -> bool {
      // (young waves leave the segment's last chunks to the older ones)
      uint32_t nk = se;
      if (!(youngest || second) ||
          __builtin_amdgcn_readfirstlane(__atomic_load_n(&next_chunk, __ATOMIC_RELAXED)) +
                  (youngest ? nwaves : nwaves / 2u) < se)
        nk = grab_chunk(&next_chunk, lane);
      nk = __builtin_amdgcn_readfirstlane(nk);  // wave-uniform after the join
      const bool has_next = nk < se;
      Win nw = cw;
      if (has_next) {
        nw = locate(t0.x0 + (nk - i) * 512u, sv);
        if (nw.fast) issue_raw<CP>(nw, sv, lane, nxt);
      }

      // ---- collide: LDS image first, the rest into the wave's queue ----
      {
        const uint32_t x8 = cw.xs + 8u * lane;
        const bool slow = __builtin_amdgcn_readfirstlane(cw.fast) == 0u;
        if (p.C != 0) {
          uint4 w0 = make_uint4(x8 >> 2, t, sv.rid, 0u);
          uint4 w1 = make_uint4((x8 >> 2) + 1u, t, sv.rid, 0u);
          decide_eight<PATCH, FIXED>(w0, w1, key, cur.m, cur.z, cur.p, lv, queue, ovr, F, slow, x8, L,
                              cw.xs);
        } else {
          queue_saturated<PATCH>(cur.m, cur.z, cur.p, queue, ovr, F, slow, x8, L, cw.xs);
        }
        if constexpr (PATCH) {
          if (F) {
            patch_chunk<GAL, FIXED>(queue, over, F, lane, cw.xs, sv, lv, p, a.tab, a.err, cur.m,
                             cur.z, cur.p);
            F = 0;
          }
        }
      }

      // ---- store ----
      if (cw.fast) {
        const uint32_t vo = 16u * lane;
        bstore4<CP>(rs, vo, 2u * cw.sm, cur.m);
        bstore4<CP>(rs, vo, ab + 2u * cw.xs, cur.z);
        bstore4<CP>(rs, vo, 2u * ab + 2u * cw.sp, cur.p);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t x = cw.xs + 8u * lane + e;
          if (x < L) {
            uint32_t pm = x + tm;
            pm -= (pm >= L) ? L : 0u;
            const uint32_t pp = x >= tm ? x - tm : x + L - tm;
            bstore2(rs, 2u * pm, 0u, get16(cur.m, e));
            bstore2(rs, 2u * x, ab, get16(cur.z, e));
            bstore2(rs, 2u * pp, 2u * ab, get16(cur.p, e));
          }
        }
      }
      // ---- the next chunk's windows ----
      if (has_next) chunk_fill(nw, nxt, sv, lane);
      cw = nw;
      k = nk;
      // At most kDrainAt draws stay queued, so the next chunk's 64 x 8
      // always fit; kDrainChunk resolves every chunk's draws while its lines
      // are still in the L2 (kDrainPatch has none left here).
      if (!PATCH && has_next && F > (MODE == kDrainChunk ? 0u : kDrainAt)) {
        drain_queue<GAL>(queue, over, F, lane, sv, p, a.tab, a.err);
        F = 0;
      }
      return has_next;
    };
    if (k < se) {
      Raw rb;
      chunk_fill(cw, cr, sv, lane);
      while (one(cr, rb) && one(rb, cr)) {
      }
    }
    i = se;
  }
  // With a ticket, the last block of the launch advances t of every slot in
  // the launch.  Every block has consumed its loads of t before it takes its
  // ticket (the values shaped its work), so nothing reads the new value
  // during this launch; the next launch sees it through the kernel boundary.
  if (!a.ticket) return;
  uint32_t &last = ctl[1];
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(a.ticket, 1u) == gridDim.x - 1u;
  __syncthreads();
  if (last) {
    for (uint32_t k = threadIdx.x; k < a.n_slots; k += blockDim.x) {
      const uint32_t s = a.slot_list ? a.slot_list[k] : a.slot_first + k;
      a.tslot[s] += 1u;
    }
    if (threadIdx.x == 0) atomicExch(a.ticket, 0u);
  }
}

// n_i(x, 0) ~ Poisson(f_i^eq): one Philox call per site (counter (x, 0,
// replica, 1)), words 0, 1, 2 for i = -1, 0, +1, inverse CDF over the host's
// quantised thresholds.  t must be 0, so physical = logical order.
__global__ void __launch_bounds__(256) k_init_poisson(
    uint16_t *__restrict__ state, const SlotDev *__restrict__ slots,
    const TileDev *__restrict__ tiles, uint32_t tile_sites, const PoisDesc *__restrict__ desc,
    const uint32_t *__restrict__ pool, uint64_t seed, uint32_t *err) {
  const TileDev tile = tiles[blockIdx.x];
  const SlotDev sl = slots[tile.slot];
  const uint2 key = make_uint2((uint32_t)seed, (uint32_t)(seed >> 32));
  const uint32_t end = min(sl.L, tile.x0 + tile_sites);
  for (uint32_t x = tile.x0 + threadIdx.x; x < end; x += blockDim.x) {
    const uint4 w = philox10(make_uint4(x, 0u, sl.rid, 1u), key);
#pragma unroll
    for (uint32_t i = 0; i < 3; ++i) {
      const PoisDesc d = desc[3u * tile.slot + i];
      const uint32_t n = d.k_first + count_le(pool + d.off, d.nthr, word_of(w, i));
      if (n > 65535u) atomicOr(err, kErrOverflow);
      state[sl.off + (uint64_t)i * sl.stride + x] = (uint16_t)n;
    }
  }
}

__global__ void __launch_bounds__(256) k_init_counts(uint16_t *__restrict__ state,
                                                     const SlotDev *__restrict__ slots,
                                                     const TileDev *__restrict__ tiles,
                                                     uint32_t tile_sites,
                                                     const uint16_t *__restrict__ counts) {
  const TileDev tile = tiles[blockIdx.x];
  const SlotDev sl = slots[tile.slot];
  const uint32_t end = min(sl.L, tile.x0 + tile_sites);
  const uint16_t *src = counts + 3ull * sl.dense;
  for (uint32_t x = tile.x0 + threadIdx.x; x < end; x += blockDim.x)
#pragma unroll
    for (uint32_t i = 0; i < 3; ++i)
      state[sl.off + (uint64_t)i * sl.stride + x] = src[(uint64_t)i * sl.L + x];
}

__global__ void k_add_t(uint32_t *tslot, uint32_t slot_first, uint32_t n, uint32_t add) {
  for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
    tslot[slot_first + k] += add;
}
__global__ void k_add_each(uint32_t *tslot, const uint32_t *add, uint32_t n) {
  for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
    tslot[k] += add[k];
}
// Bound by the host link's latency: one launch for all pieces of an update
// (blockIdx.y), read where the host wrote them, in place of a copy of its
// own for each (about 7 us and 10 us of waiting between queues).
__global__ void __launch_bounds__(256) k_uploads(Uploads u) {
  const auto p = u.piece[blockIdx.y];
  const uint64_t n = p.bytes / 4u, step = (uint64_t)gridDim.x * blockDim.x;
  const uint32_t *const src = static_cast<const uint32_t *>(p.src);
  uint32_t *const dst = static_cast<uint32_t *>(p.dst);
  for (uint64_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) dst[i] = src[i];
}
__global__ void k_set_t(uint32_t *tslot, const uint32_t *slot_list, uint32_t n, uint32_t value) {
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) tslot[slot_list[i]] = value;
}

// Occupation-number histograms.  Each block takes a contiguous run of tiles
// (tiles are ordered by slot), reads every velocity array in physical order
// (a marginal histogram does not depend on which site an element belongs
// to), bins in LDS, and adds each non-empty bin to the slot's global row with
// one 64-bit atomic whenever the run moves to another slot or ends.
__global__ void __launch_bounds__(256) k_histogram(
    const uint16_t *__restrict__ state, const SlotDev *__restrict__ slots,
    const TileDev *__restrict__ tiles, uint32_t n_tiles, uint32_t tile_sites, uint32_t n_bins,
    unsigned long long *__restrict__ hist) {
  extern __shared__ uint32_t bins[];  // [3][n_bins]
  const uint32_t per = (n_tiles + gridDim.x - 1u) / gridDim.x;
  const uint32_t t_begin = blockIdx.x * per, t_end = min(n_tiles, t_begin + per);
  if (t_begin >= t_end) return;
  const uint32_t nb3 = 3u * n_bins, top = n_bins - 1u;
  for (uint32_t j = threadIdx.x; j < nb3; j += blockDim.x) bins[j] = 0u;
  uint32_t cur = tiles[t_begin].slot;
  auto flush = [&](uint32_t slot) {
    __syncthreads();
    unsigned long long *row = hist + (uint64_t)slot * nb3;
    for (uint32_t j = threadIdx.x; j < nb3; j += blockDim.x) {
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
    const TileDev tile = tiles[t];
    if (tile.slot != cur) {
      flush(cur);
      cur = tile.slot;
    }
    const SlotDev sl = slots[tile.slot];
    const uint32_t end = min(sl.L, tile.x0 + tile_sites);
    for (uint32_t x = tile.x0 + threadIdx.x; x < end; x += blockDim.x) {
#pragma unroll
      for (uint32_t i = 0; i < 3u; ++i) {
        const uint32_t n = state[sl.off + (uint64_t)i * sl.stride + x];
        atomicAdd(&bins[i * n_bins + min(n, top)], 1u);
      }
    }
  }
  flush(cur);
}

}  // namespace

// Sets the dynamic LDS limit of the twelve instantiations for this block size
// and returns the smallest of their occupancies.
template <int MAXT, bool GAL, int MODE, bool FIXED>
static hipError_t occupancy_one(uint32_t threads, uint32_t lds, int &blocks) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_step<MAXT, GAL, MODE, FIXED>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e) return e;
  int b = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_step<MAXT, GAL, MODE, FIXED>, (int)threads, lds);
  blocks = std::min(blocks, b);
  return e;
}
template <int MAXT, bool GAL>
static hipError_t occupancy_modes(uint32_t threads, uint32_t lds, int &blocks) {
  hipError_t e = occupancy_one<MAXT, GAL, kDrainDeferred, true>(threads, lds, blocks);
  if (!e) e = occupancy_one<MAXT, GAL, kDrainChunk, true>(threads, lds, blocks);
  if (!e) e = occupancy_one<MAXT, GAL, kDrainPatch, true>(threads, lds, blocks);
  if (!e) e = occupancy_one<MAXT, GAL, kDrainDeferred, false>(threads, lds, blocks);
  if (!e) e = occupancy_one<MAXT, GAL, kDrainChunk, false>(threads, lds, blocks);
  if (!e) e = occupancy_one<MAXT, GAL, kDrainPatch, false>(threads, lds, blocks);
  return e;
}
template <int MAXT>
static hipError_t occupancy_of(uint32_t threads, uint32_t lds, int &blocks) {
  blocks = 1 << 30;
  hipError_t e = occupancy_modes<MAXT, false>(threads, lds, blocks);
  if (!e) e = occupancy_modes<MAXT, true>(threads, lds, blocks);
  return e;
}

uint32_t step_lds_bytes(const Schedule &sch, uint32_t image_bytes) {
  return (image_bytes + 15u) / 16u * 16u + (sch.threads / 64u) * kWaveLdsBytes + 16u;
}

// Blocks of up to 512 threads may use up to 256 VGPRs per lane.
hipError_t step_occupancy(const Schedule &sch, uint32_t lds_bytes, uint32_t n_cu,
                          uint32_t &max_blocks) {
  int b = 0;
  if (sch.groups != 1) return hipErrorInvalidValue;
  const uint32_t lds = step_lds_bytes(sch, lds_bytes);
  hipError_t e = sch.threads <= 512 ? occupancy_of<512>(sch.threads, lds, b)
                                    : occupancy_of<1024>(sch.threads, lds, b);
  if (e) return e;
  if (b < 1) return hipErrorInvalidConfiguration;
  max_blocks = (uint32_t)b * n_cu;
  return hipSuccess;
}

template <int MAXT, bool GAL, bool FIXED>
static void launch_fixed(dim3 grid, dim3 block, uint32_t lds, hipStream_t s, const StepLaunch &a) {
  switch (a.p.drain) {
    case kDrainChunk: k_step<MAXT, GAL, kDrainChunk, FIXED><<<grid, block, lds, s>>>(a); break;
    case kDrainPatch: k_step<MAXT, GAL, kDrainPatch, FIXED><<<grid, block, lds, s>>>(a); break;
    default: k_step<MAXT, GAL, kDrainDeferred, FIXED><<<grid, block, lds, s>>>(a); break;
  }
}
template <int MAXT, bool GAL>
static void launch_mode(dim3 grid, dim3 block, uint32_t lds, hipStream_t s, const StepLaunch &a) {
  if (images_fixed(a.p.C)) launch_fixed<MAXT, GAL, true>(grid, block, lds, s, a);
  else launch_fixed<MAXT, GAL, false>(grid, block, lds, s, a);
}

hipError_t launch_step(const Schedule &sch, hipStream_t s, const StepLaunch &a) {
  if (a.n_tiles == 0) return hipSuccess;
  dim3 grid(std::max<uint32_t>(1, std::min(a.n_tiles, a.max_blocks))), block(sch.threads);
  const uint32_t lds = step_lds_bytes(sch, a.lds_bytes);
  if (sch.groups != 1) return hipErrorInvalidValue;
  if (a.p.drain > kDrainPatch) return hipErrorInvalidValue;
  const bool small = sch.threads <= 512;
  if (a.p.galilean) {
    if (small) launch_mode<512, true>(grid, block, lds, s, a);
    else launch_mode<1024, true>(grid, block, lds, s, a);
  } else {
    if (small) launch_mode<512, false>(grid, block, lds, s, a);
    else launch_mode<1024, false>(grid, block, lds, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_init_poisson(hipStream_t s, uint16_t *state, const SlotDev *slots,
                               const uint32_t *, const TileDev *tiles, uint32_t n_tiles,
                               uint32_t tile_sites, const PoisDesc *desc, const uint32_t *pool,
                               uint64_t seed, uint32_t *err) {
  if (n_tiles == 0) return hipSuccess;
  k_init_poisson<<<n_tiles, 256, 0, s>>>(state, slots, tiles, tile_sites, desc, pool, seed, err);
  return hipGetLastError();
}

hipError_t launch_init_counts(hipStream_t s, uint16_t *state, const SlotDev *slots,
                              const TileDev *tiles, uint32_t n_tiles, uint32_t tile_sites,
                              const uint16_t *counts) {
  if (n_tiles == 0) return hipSuccess;
  k_init_counts<<<n_tiles, 256, 0, s>>>(state, slots, tiles, tile_sites, counts);
  return hipGetLastError();
}

hipError_t launch_histogram(hipStream_t s, const uint16_t *state, const SlotDev *slots,
                            const TileDev *tiles, uint32_t n_tiles, uint32_t tile_sites,
                            uint32_t n_bins, unsigned long long *hist) {
  if (n_tiles == 0) return hipSuccess;
  const uint32_t blocks = std::min<uint32_t>(n_tiles, 2048u);
  k_histogram<<<blocks, 256, 3u * n_bins * sizeof(uint32_t), s>>>(state, slots, tiles, n_tiles,
                                                                  tile_sites, n_bins, hist);
  return hipGetLastError();
}

hipError_t launch_add_t(hipStream_t s, uint32_t *tslot, uint32_t slot_first, uint32_t n,
                        uint32_t add) {
  if (n == 0 || add == 0) return hipSuccess;
  k_add_t<<<std::min<uint32_t>(64, (n + 255) / 256), 256, 0, s>>>(tslot, slot_first, n, add);
  return hipGetLastError();
}

hipError_t launch_add_each(hipStream_t s, uint32_t *tslot, const uint32_t *add, uint32_t n) {
  if (n == 0) return hipSuccess;
  k_add_each<<<std::min<uint32_t>(64, (n + 255) / 256), 256, 0, s>>>(tslot, add, n);
  return hipGetLastError();
}

hipError_t launch_uploads(hipStream_t s, const Uploads &u) {
  if (u.n == 0) return hipSuccess;
  if (u.n > kUploads) return hipErrorInvalidValue;
  k_uploads<<<dim3(32, u.n), 256, 0, s>>>(u);
  return hipGetLastError();
}

hipError_t launch_set_t(hipStream_t s, uint32_t *tslot, const uint32_t *slot_list, uint32_t n,
                        uint32_t value) {
  if (n == 0) return hipSuccess;
  k_set_t<<<1, 256, 0, s>>>(tslot, slot_list, n, value);
  return hipGetLastError();
}

}  // namespace mclg
