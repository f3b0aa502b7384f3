// How the steps of a context's lattices are laid out for the kernels that
// hold sites in registers (host side): the parts each block takes, and which
// kernel, how many sites per lane and how many steps per launch a call takes.
#pragma once
#include <cstdint>
#include <vector>

#include "device.h"

namespace mclg {

constexpr uint32_t kPlanBlocks = 256;      // blocks of a tile launch, at most
constexpr uint32_t kMaxStrips = 4 * kPlanBlocks;
inline uint64_t max_units(uint32_t n) { return (uint64_t)n + kMaxStrips; }

// Lattices of fewer sites never go in tiles (a tile with its extra sites must
// be shorter than its lattice); beside longer ones they take the ring kernel.
constexpr uint32_t kMinTiled = 512;

// The time of a site of a lattice whose image decides `coverage` of them, that
// of one with all decided as 1 (2^24 sites, Q = 4, us per step: all 22.4, all
// but 0.3 % 27.5, 2 % 34.7, 11 % 42; most of it is paid for the first few of a
// wave's step).
inline float site_cost(double coverage) {
  const double m = coverage < 1.0 ? 1.0 - coverage : 0.0;
  return (float)(1.0 + 0.95 * m / (m + 0.01));
}

// How unevenly a SIMD's waves share tiles (see k_tile): best, with many tiles,
// at 12 to 13 where all sites are decided, 10 to 11 with 0.3 % undecided, 8
// with 11 %.
inline uint32_t image_skew(double coverage) {
  return (uint32_t)(13.5 - 4.5 * ((double)site_cost(coverage) - 1.0));
}

// The units of the tile kernel: every lattice of at least kMinTiled sites,
// whole or in equal parts, dealt to the blocks longest first (cost: of a site
// of each lattice, from 1 to 2; null: 1).
struct UnitPlan {
  uint32_t n_long = 0;           // such lattices
  std::vector<UnitDev> units;
  std::vector<uint32_t> first;   // blocks + 1
  std::vector<StripDev> strips;
};
UnitPlan plan_units(const uint64_t *L, uint32_t n, uint32_t blocks, const float *cost = nullptr);

// One way to take steps: the kernel, its sites per lane (4 Q) and, for the
// tiles, the sites on each side (steps per launch, at most).
struct RegWay {
  enum Kind : uint32_t { kNone = 0, kRing, kTile } kind = kNone;
  uint32_t Q = 0, kh = 0, team = 0;
  uint32_t most = 0;                  // steps per launch, at most
  bool logs = false;                  // whether a launch can sum logs
  double launch_us = 0, step_us = 0;  // per launch and per step, estimated
  // Against one step per launch: the fewest steps a launch is taken for, and
  // the estimates with what all ways share and what few steps don't hide
  // (few_in_us: divided by the launch's steps).
  uint32_t least = 1;
  double few_launch_us = 0, few_in_us = 0, few_step_us = 0;
};

// Whether a wave's step of 1536 sites leaves more undecided than its queue of
// 64 takes, for an image that decides `coverage` of them.
inline bool crowded_image(double coverage) { return coverage < 1.0 - 64.0 / 1536.0; }

// The ways open to a context, with their estimated times; one_image: all
// lattices share one; crowded: the share of the sites in lattices of crowded
// images.
std::vector<RegWay> plan_ways(const UnitPlan &plan, const uint64_t *L, uint32_t n, uint32_t blocks,
                              bool one_image, bool galilean, bool fixed, double crowded,
                              const float *cost = nullptr);

// One step per launch of the kernels that keep the state in memory, per step:
// as the ways' estimates were fitted beside it, and with the sites the images
// don't decide and the lattices' number.
struct SingleStep {
  double us = 0, few_us = 0;
};
// missed: the share of the sites whose draws the images don't decide.
SingleStep single_step(uint64_t sites, uint32_t n, bool one_image, double missed, bool fixed);

// The quickest way for `steps` steps, or nullptr when one step per launch is
// quicker.
const RegWay *pick_way(const std::vector<RegWay> &ways, uint64_t steps, const SingleStep &single);

// The quickest way for n_logs times `every` steps with the moments of `sites`
// sites after each, or nullptr where it is quicker to take every interval by
// itself and sum its state in memory.
const RegWay *pick_log_way(const std::vector<RegWay> &ways, uint64_t every, uint64_t n_logs, uint64_t sites,
                           uint32_t n_modes, bool digest, const SingleStep &single);

}  // namespace mclg
