// Launching a way of taking several steps on sites held in registers, for a
// context's replicas or a server's resident jobs.
#pragma once

#include "device.h"
#include "regplan.h"

namespace mclg {

// Device copies of a plan's lists, and its strips' counts.
struct RegBufs {
  const uint32_t *order = nullptr;  // the lattices' slots, longest first
  uint32_t n = 0;
  const UnitDev *units = nullptr;
  const uint32_t *first = nullptr;
  const StripDev *strips = nullptr;
  uint16_t *strip_data = nullptr;
  const uint32_t *limit = nullptr;  // by slot, or null (see RingLaunch)
};

// Records per log and lattice.
inline uint32_t log_records(const RegWay &w, const UnitPlan &plan) {
  return w.kind == RegWay::kTile ? ((uint32_t)plan.first.size() - 1u) * kRegWaves : w.team ? 1u : kRegWaves;
}

// `steps` steps (at most w.most) of every lattice in one launch of way `w`,
// with the logs lg.first, ... of them.
inline hipError_t launch_way(hipStream_t s, const StepLaunch &a, const RegWay &w, const UnitPlan &plan,
                             const RegBufs &b, uint32_t steps, const RegLog &lg) {
  RingLaunch r;
  r.steps = steps;
  r.limit = b.limit;
  if (w.kind == RegWay::kRing) {
    r.order = b.order;
    r.n = b.n;
    r.team = w.team;
    r.log = lg;
    r.log.stride = log_records(w, plan);
    r.log.hold = w.team ? 0u : 256u * w.Q;
    return launch_ring(s, a, r, w.Q, kRegWaves);
  }
  TileLaunch tl;
  tl.units = b.units;
  tl.unit_first = b.first;
  tl.strips = b.strips;
  tl.strip_data = b.strip_data;
  tl.n_strips = (uint32_t)plan.strips.size();
  tl.kh = w.kh;
  tl.steps = steps;
  tl.limit = b.limit;
  tl.log = lg;
  tl.log.stride = log_records(w, plan);
  hipError_t e = launch_tiles(s, a, tl, w.Q, kRegWaves, (uint32_t)plan.first.size() - 1, b.order);
  if (!e && plan.n_long < b.n) {  // the lattices too short for tiles, last in the order
    r.order = b.order + plan.n_long;
    r.n = b.n - plan.n_long;
    e = launch_ring(s, a, r, 2, kRegWaves);
  }
  return e;
}

}  // namespace mclg
