// Device-side data structures and launchers of the MCLG library (gfx950).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace mclg {

// One simulated lattice ("slot").  Its state is three uint16 arrays of
// `stride` elements starting at element `off` of the state buffer:
// n_-1, n_0, n_+1.  In-place shifted layout: logical n_+1(x, t) is stored at
// physical (x - t) mod L, n_-1(x, t) at (x + t) mod L, n_0(x) at x, so that
// streaming costs nothing and every element is read and written by exactly
// one site per step.  With MCLG_FLAG_NO_STREAM the layout is unshifted.
struct SlotDev {
  uint64_t off = 0;      // element offset of the n_-1 array in the state buffer
  uint64_t dense = 0;    // packed site offset (init counts, twiddles)
  uint32_t L = 0;        // sites
  uint32_t stride = 0;   // elements per array (L rounded up to 128)
  uint32_t rid = 0;      // RNG replica identity
  uint32_t pad = 0;
};

// A chunk of 512 sites of one slot (the last chunk of a slot may be short).
struct TileDev {
  uint32_t slot = 0;     // slot index
  uint32_t x0 = 0;       // first site (multiple of 512)
  uint32_t next = 0;     // index of the first chunk after this slot's run of chunks
  uint32_t pad = 0;
};

// Queued draws a wave may keep between chunks (the LDS queue and 32 more).
constexpr uint32_t kDrainAt = 64 + 32;

// When the draws the LDS image cannot decide are resolved (from the exact
// global rows), per wave:
//   kDrainDeferred: queued until more than kDrainAt wait, then resolved after
//     the chunk's store and written with 2-byte stores into the lines the
//     chunks stored before;
//   kDrainChunk: the same after every chunk's store;
//   kDrainPatch: before the chunk's store -- the exact outcomes go into the
//     chunk's registers, so the chunk's 16-byte stores write final values and
//     nothing is written twice.
enum : uint32_t { kDrainDeferred = 0, kDrainChunk = 1, kDrainPatch = 2 };

struct StepParams {
  uint64_t seed = 0;
  int32_t C = 0;
  uint32_t lam_p = 1, lam_q = 1;
  uint32_t n_max = 0;
  uint32_t no_stream = 0;
  uint32_t tile_sites = 512;
  uint32_t galilean = 0;  // per-site lambda (see collide_direct)
  uint32_t drain = kDrainDeferred;
};

// Deferred 2-byte writes land in lines the chunks stored long before.  While
// a launch's state fits the 256 MB Infinity Cache those lines are still
// cached and the writes are cheap; a larger state has left the caches by
// then, and partial-line writes into it are slow, so each chunk's draws are
// resolved before its store.
constexpr uint64_t kCachedStateBytes = 256ull << 20;
inline uint32_t auto_drain(uint64_t launch_state_bytes) {
  return launch_state_bytes > kCachedStateBytes ? kDrainPatch : kDrainDeferred;
}

// Index of the collision row of a site with N particles, n0 = b of them at
// rest and a = min(n_-1, n_+1): rows are ordered by N, then s = N - b, then a
// = 0 .. s / 2, so floor((s + 1)^2 / 4) rows of N precede those of s, and
// sum_{k <= N + 1} floor(k^2 / 4) = floor((N + 1)(N + 3)(2 N + 1) / 24) rows
// those of N.  (In 32 bits for N <= 1023.)
__host__ __device__ inline uint32_t collision_row(uint32_t N, uint32_t b, uint32_t a) {
  const uint32_t s1 = N - b + 1u;
  return (N + 1u) * (N + 3u) * (2u * N + 1u) / 24u + ((s1 * s1) >> 2) + a;
}

// uint16 values per row of the 64-byte copy of the collision rows: k_first
// and the top 15 bits of up to 31 thresholds.
constexpr uint32_t kRow16 = 32;

struct TableDev {
  const uint2 *rowdesc = nullptr;
  const uint32_t *thr = nullptr;
  const uint4 *row16 = nullptr;  // rows of kRow16 uint16 (64 bytes), or null
  uint32_t row_words = 16;       // words of such a row that hold thresholds: 12 or 16
  uint32_t pad = 0;
};

// Where a slot's LDS image lives in the image pool (see LdsImage).
struct ImageDesc {
  uint64_t off = 0;        // byte offset in the image pool (16-byte aligned)
  uint32_t bytes = 0;      // every slot has one (at least the two special slots)
  uint32_t dir_bytes = 0;
  uint32_t dim_a = 0, dim_c = 0, b_lo = 0, nb = 0;
  uint32_t fixed = 0;      // records with the window of moves around none (see LdsImage)
  uint32_t skew = 0;       // of a SIMD's waves in a tile launch (see k_tile), at most 21
};

struct PoisDesc {
  uint32_t off = 0;      // offset in the threshold pool
  uint32_t k_first = 0;
  uint32_t nthr = 0;     // q - 1
  uint32_t pad = 0;
};

// Launch configuration of the fused stream+collide kernel.
struct Schedule {
  uint32_t groups = 1;       // chunks of 8 sites per lane (must be 1)
  uint32_t threads = 1024;   // threads per block
  uint32_t lds_budget = 160 * 1024;  // bytes of collision image per block (at most)
  uint32_t tile_sites() const { return 512; }  // one chunk: 64 lanes x 8 sites
};

// Every field has an initialiser, so that a launch record built field by
// field never carries an indeterminate value.
struct StepLaunch {
  uint16_t *state = nullptr;
  const SlotDev *slots = nullptr;
  uint32_t *tslot = nullptr;
  const TileDev *tiles = nullptr;
  uint32_t n_tiles = 0;
  const uint32_t *slot_list = nullptr;  // slots advanced by this launch, or null for a range
  uint32_t slot_first = 0, n_slots = 0;
  // With `ticket` set, the launch's last block advances tslot of the launch's
  // slots by one; without it the slots' step is tslot + t_off and tslot is
  // advanced later (launch_add_t), which saves the end-of-launch ticket.
  uint32_t *ticket = nullptr, *err = nullptr;
  uint32_t t_off = 0;
  // A launch over one slot's tiles (0 .. n_tiles - 1 from x = 0) carries the
  // slot's descriptors itself, so that its blocks start without dependent
  // loads: single = 1, slot slot_first, image im1, slot sl1.
  uint32_t single = 0;
  ImageDesc im1;
  SlotDev sl1;
  TableDev tab;
  StepParams p;
  const ImageDesc *images = nullptr;  // per slot
  const uint8_t *image_pool = nullptr;
  uint4 *overflow = nullptr;          // kOverflowPerWave entries per resident wave
  uint32_t lds_bytes = 0;             // LDS per block for the image (largest image, 16-byte
                                      // multiple); the per-wave miss queues follow it
  uint32_t max_blocks = 1;            // persistent grid size
};

hipError_t launch_step(const Schedule &sch, hipStream_t s, const StepLaunch &a);

// Largest lattice (sites per replica or job): the step kernel addresses a
// slot's three arrays (6 bytes per site, 256-byte padded) with 32-bit byte
// offsets.
constexpr uint64_t kMaxSites = 1ull << 29;
constexpr uint32_t kQueue = 64;  // LDS queue entries (16 bytes) per wave
static_assert(kDrainAt == kQueue + 32, "drain threshold follows the LDS queue");
// per-wave LDS after the image: the queue of undecided draws
constexpr uint32_t kWaveLdsBytes = kQueue * 16;
// Entries of the global overflow area per wave (the queue continues there
// when its LDS part is full: up to 32 entries beyond it plus one chunk's
// 512 sites), and the number of waves the overflow region is sized for (all
// waves that can be resident on a 256-CU device).
constexpr uint32_t kOverflowPerWave = 576;
constexpr uint32_t kOverflowWaves = 256 * 32;
constexpr uint64_t kOverflowBytes = (uint64_t)kOverflowPerWave * kOverflowWaves * 16;

// Persistent grid size: resident blocks per CU for this LDS footprint x CUs.
hipError_t step_occupancy(const Schedule &sch, uint32_t lds_bytes, uint32_t n_cu,
                          uint32_t &max_blocks);
// Dynamic LDS of one block: image (rounded to 16 bytes) + miss queues.
uint32_t step_lds_bytes(const Schedule &sch, uint32_t image_bytes);

// ---- Steps on sites held in registers (kernels_reg.hip) -----------------
// Logs: the moments (mclg_moments_t) of the states after steps first, first +
// every, ... (n of them) of a launch.  Every wave writes one record of
// kMom3Rec values per log and lattice, at records + ((log x lattices +
// lattice) x stride + wave) kMom3Rec; their sums go to out, in the order of
// mclg_step_log.  hold: sites per wave, where a lattice has that many waves'
// records (0: all `stride`).
struct RegLog {
  uint32_t first = 0, every = 0, n = 0;
  uint32_t n_modes = 0, digest = 0, stride = 0, hold = 0, pad = 0;
  const int32_t *tw = nullptr;
  unsigned long long *records = nullptr;
  long long *out = nullptr;
};
// Ring: lattices order[0 .. n) that fit a block's registers, `steps` steps
// in one launch.  A wave holds up to 256 Q sites.  team = 0: a block per
// lattice; team = k: k lattices of at most 256 Q sites per block, a wave
// each, all with the same image.
struct RingLaunch {
  const uint32_t *order = nullptr;  // slots
  uint32_t n = 0, team = 0, steps = 0;
  const uint32_t *limit = nullptr;  // by slot: steps of the launch that it takes (null: all)
  RegLog log;
};
// Tiles: block b advances units[unit_first[b] .. unit_first[b + 1]), each a
// whole lattice (split = 0: x0 = 0, x1 = L) or a part of one between two
// strips el and er, `steps` <= kh steps (kh - 8 when some lattice's sites are
// no multiple of 8: the positions after its last site take their place).  x0, and x1 unless it is L, are
// multiples of 8, and a part holds at least kh sites.
struct UnitDev {
  uint32_t slot = 0, x0 = 0, x1 = 0, split = 0, el = 0, er = 0;
};
// The boundary after the part of `slot` that ends at x.
struct StripDev {
  uint32_t slot = 0, x = 0;
};
constexpr uint32_t kMaxHalo = 128;  // kh, at most
struct TileLaunch {
  const UnitDev *units = nullptr;
  const uint32_t *unit_first = nullptr;
  const StripDev *strips = nullptr;
  uint16_t *strip_data = nullptr;   // n_strips x 3 x 2 kh
  uint32_t n_strips = 0, kh = 0, steps = 0;
  const uint32_t *limit = nullptr;  // as in RingLaunch
  RegLog log;                       // one lattice only
};
constexpr uint32_t kRingExchangeBytes = 128;
constexpr uint32_t kRegWaves = 16;  // waves per block
// Whether the collision images of C hold fixed records (see LdsImage).
constexpr bool images_fixed(int32_t C) { return C >= 0 && C <= 20; }
// Whether the kernels exist for 4 Q sites per lane and these rules.
bool reg_has(uint32_t Q, bool galilean, bool fixed, bool logs);
uint32_t reg_lds_bytes(uint32_t image_bytes, uint32_t waves);
// Allows the kernels the LDS of a 16-wave block with images of image_bytes.
hipError_t reg_setup(uint32_t image_bytes);
hipError_t launch_ring(hipStream_t s, const StepLaunch &a, const RingLaunch &rl, uint32_t Q,
                       uint32_t waves);
hipError_t launch_tiles(hipStream_t s, const StepLaunch &a, const TileLaunch &tl, uint32_t Q,
                        uint32_t waves, uint32_t grid, const uint32_t *order);

hipError_t launch_init_poisson(hipStream_t s, uint16_t *state, const SlotDev *slots,
                               const uint32_t *tslot, const TileDev *tiles, uint32_t n_tiles,
                               uint32_t tile_sites, const PoisDesc *desc, const uint32_t *pool,
                               uint64_t seed, uint32_t *err);

hipError_t launch_init_counts(hipStream_t s, uint16_t *state, const SlotDev *slots,
                              const TileDev *tiles, uint32_t n_tiles, uint32_t tile_sites,
                              const uint16_t *counts);

// hist[(slot * 3 + i) * n_bins + min(n_i, n_bins - 1)] += 1 over every site
hipError_t launch_histogram(hipStream_t s, const uint16_t *state, const SlotDev *slots,
                            const TileDev *tiles, uint32_t n_tiles, uint32_t tile_sites,
                            uint32_t n_bins, unsigned long long *hist);

// tslot[slot_first + i] += add for i < n
hipError_t launch_add_t(hipStream_t s, uint32_t *tslot, uint32_t slot_first, uint32_t n,
                        uint32_t add);
// tslot[i] += add[i].
hipError_t launch_add_each(hipStream_t s, uint32_t *tslot, const uint32_t *add, uint32_t n);
// Copies of `n` pieces of pinned host memory (whole words) to device memory.
constexpr uint32_t kUploads = 24;
struct Uploads {
  struct {
    void *dst;
    const void *src;
    uint64_t bytes;
  } piece[kUploads];
  uint32_t n = 0;
};
hipError_t launch_uploads(hipStream_t s, const Uploads &u);
hipError_t launch_set_t(hipStream_t s, uint32_t *tslot, const uint32_t *slot_list, uint32_t n,
                        uint32_t value);

// ---- D2Q9 --------------------------------------------------------------
// One replica: nine uint16 arrays of `stride` elements from `off`; logical
// n_i(x, y, t) lives at physical ((x - vx t) mod Lx, (y - vy t) mod Ly),
// element y Lx + x, so streaming is free as for D1Q3.
struct Rep9 {
  uint64_t off;
  uint32_t Lx, Ly, S, stride;
  uint32_t rid, pad;
};
struct Tile9 {
  uint32_t rep, s0;  // replica, first site (multiple of kTileSites9)
  uint32_t x0;       // s0 mod Lx
};
constexpr uint32_t kTileSites9 = 256;
// Collision rules, per ordered source pair (v1, v2), kRule9Words uint32:
// words 0-3 the cumulative integer weights of the (up to four) targets, D
// where there is none; words 4-8 the change of the nine counts for target
// q = #{cumulative weights <= u} (word 4 + q; q = number of targets means no
// change), 3 bits per velocity i at bit 3i holding 2 + the change; 9-11 pad.
constexpr uint32_t kRule9Words = 12;
struct Step9 {
  uint16_t *state;
  const Rep9 *reps;
  const Tile9 *tiles;
  const uint32_t *rules;
  uint32_t *err;
  uint64_t seed;
  uint64_t t;          // steps taken (the RNG counter uses its low 32 bits)
  uint32_t D, no_stream;
  uint32_t Dq;         // D divided by the greatest common divisor of it and all weights
  int32_t C;
  uint32_t first_table;  // of the rules that a block begins with: 1 bytes, 2 halves (both for
                         // Dq <= kRule9MaxPacked only), 3 any
};
hipError_t launch_step9(hipStream_t s, const Step9 &a, uint32_t n_tiles);
// `steps` steps of lattices of up to kBlockSites9 sites in one launch.
constexpr uint32_t kBlockSites9 = 512;
hipError_t launch_steps9(hipStream_t s, const Step9 &a, uint32_t n_reps, uint32_t max_sites,
                         uint32_t steps);
hipError_t launch_init9_poisson(hipStream_t s, uint16_t *state, const Rep9 *reps,
                                const Tile9 *tiles, uint32_t n_tiles, const PoisDesc *desc,
                                const uint32_t *pool, uint64_t seed, uint32_t *err);
hipError_t launch_init9_counts(hipStream_t s, uint16_t *state, const Rep9 *reps,
                               const Tile9 *tiles, uint32_t n_tiles, const uint64_t *dense,
                               const uint16_t *counts, uint32_t *full);  // += tiles with N >= 128
hipError_t launch_histogram9(hipStream_t s, const uint16_t *state, const Rep9 *reps,
                             const Tile9 *tiles, uint32_t n_tiles, uint32_t n_bins,
                             unsigned long long *hist);
}  // namespace mclg
