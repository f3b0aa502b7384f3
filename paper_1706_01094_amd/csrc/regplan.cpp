#include "regplan.h"

#include <algorithm>
#include <cmath>
#include <numeric>

namespace mclg {

namespace {
constexpr uint64_t kMinPart = 256;  // work of a block, at least, in sites of cost 1
static_assert(kMaxHalo % 8 == 0, "a part of kMaxHalo sites ends at a multiple of 8");
}  // namespace

UnitPlan plan_units(const uint64_t *L, uint32_t n, uint32_t blocks, const float *cost) {
  UnitPlan P;
  blocks = std::min(blocks, kPlanBlocks);
  // the work of s sites of lattice r, in sites of cost 1
  auto weigh = [&](uint32_t r, uint64_t s) { return cost ? (uint64_t)((double)s * cost[r]) : s; };
  uint64_t total = 0;
  for (uint32_t r = 0; r < n; ++r) {
    if (L[r] < kMinTiled) continue;
    total += weigh(r, L[r]);
    ++P.n_long;
  }
  const uint64_t target = std::max<uint64_t>(kMinPart, (total + blocks - 1) / blocks);
  std::vector<UnitDev> all;
  for (uint32_t r = 0; r < n; ++r) {
    if (L[r] < kMinTiled) continue;
    // a lattice of up to 5/4 of a block's share stays whole
    const uint64_t work = weigh(r, L[r]);
    uint64_t parts = 4 * work <= 5 * target ? 1 : (work + target - 1) / target;
    if (P.strips.size() + parts > kMaxStrips) parts = 1;
    // (no part is shorter than the sites on each side of a tile; parts of equal
    // work would be, where a site costs nearly 2)
    const uint64_t len = std::max<uint64_t>(kMaxHalo, ((L[r] + parts - 1) / parts + 7) / 8 * 8);
    parts = (L[r] + len - 1) / len;
    if (parts > 1 && L[r] - (parts - 1) * len < kMaxHalo) --parts;  // (the last part takes the rest)
    const uint32_t s0 = (uint32_t)P.strips.size();
    for (uint64_t j = 0; j < parts; ++j) {
      UnitDev u;
      u.slot = r;
      u.x0 = (uint32_t)(j * len);
      u.x1 = (uint32_t)(j + 1 < parts ? (j + 1) * len : L[r]);
      if (parts > 1) {
        u.split = 1;
        u.el = s0 + (uint32_t)((j + parts - 1) % parts);
        u.er = s0 + (uint32_t)j;
        P.strips.push_back(StripDev{r, u.x1});
      }
      all.push_back(u);
    }
  }
  // longest first to the block with the least (a unit's fixed cost counts as
  // 2048 sites); a block's units keep the order of the lattices, so that
  // units of one image follow each other
  std::vector<uint32_t> order(all.size());
  std::iota(order.begin(), order.end(), 0u);
  auto work = [&](uint32_t i) { return weigh(all[i].slot, all[i].x1 - all[i].x0) + 2048u; };
  std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) { return work(x) > work(y); });
  std::vector<std::pair<uint64_t, uint32_t>> heap;
  for (uint32_t b = 0; b < blocks; ++b) heap.push_back({0, b});
  auto more = [](const std::pair<uint64_t, uint32_t> &x, const std::pair<uint64_t, uint32_t> &y) { return x > y; };
  std::make_heap(heap.begin(), heap.end(), more);
  std::vector<std::vector<uint32_t>> lists(blocks);
  for (uint32_t i : order) {
    std::pop_heap(heap.begin(), heap.end(), more);
    heap.back().first += work(i);
    lists[heap.back().second].push_back(i);
    std::push_heap(heap.begin(), heap.end(), more);
  }
  for (auto &l : lists) {
    std::sort(l.begin(), l.end());
    P.first.push_back((uint32_t)P.units.size());
    for (uint32_t i : l) P.units.push_back(all[i]);
  }
  P.first.push_back((uint32_t)P.units.size());
  return P;
}

namespace {
constexpr uint64_t kCachedSites = 44ull << 20;  // whose counts the Infinity Cache holds

// Times on MI355X (us), fitted to measured steps of lattices of 256 to 2^27
// sites at rho = 50.  A wave that is alone on its SIMD takes 0.72 + 0.58 Q for
// a step of its 256 Q sites (latency); a SIMD with one or more for each of its
// four waves issues for 0.14 + 0.283 Q per tile (as dealt by k_tile), and a
// little for the end where not all have one; with fewer, 0.27 + 0.28 Q.  Both
// together take a little more than the larger of the two.
double tile_step_us(uint32_t Q, uint64_t tiles) {
  const double n = tiles > 16 ? (double)tiles / 4.0 : (double)((tiles + 3) / 4);
  const double issue = tiles > 16 ? (0.14 + 0.283 * Q) * (n + 0.3 + 0.2 * Q) : n * (0.27 + 0.28 * Q);
  const double wait = std::max(1.0, (double)tiles / 16.0) * (0.72 + 0.58 * Q);
  const double most = std::max(issue, wait), x = std::min(issue, wait) / most;
  return most * std::sqrt(std::sqrt(1.0 + x * x * x * x));
}
// A lattice in one block's registers: without the private areas and the
// extra sites, but with a barrier per step when several waves hold it.
double ring_step_us(uint32_t Q, uint32_t waves, bool together) {
  const double issue = (waves + 3) / 4 * (0.27 + 0.28 * Q), wait = 0.55 + 0.5 * Q;
  const double step = std::sqrt(std::sqrt(issue * issue * issue * issue + wait * wait * wait * wait));
  return step + (together && waves > 1 ? 0.5 + 0.1 * Q : 0.0);
}
constexpr double kRingLaunch = 5.0;   // launch, image and the sites' way in and out
// The same for the tiles; to it comes the state's way in and out, of which the
// registers of Q = 6 leave more uncovered.  Measured, us per launch at 2^20,
// 2^22, 2^24 and 2^27 sites: Q <= 4 16, 23, 45 and 125, Q = 6 19, 32, 55 and
// 200.
constexpr double kTileLaunch = 12.0;
double state_us(uint32_t Q, uint64_t sites) {
  const double s = (double)sites, most = (double)(1u << 24);
  return 1.6e-6 * std::min(s, most) + 0.9e-6 * std::max(0.0, s - most) + (Q < 6 ? 0.0 : 6.0 + 0.45e-6 * s);
}
// A launch of few steps: the state's way in and out is not covered by work,
// and the estimates' common factors (a site's cost where its image leaves more
// undecided than at density 50, and that of the kernels with other rules)
// count against a launch per step, which they are not in.  Us per launch
// measured (and a launch per step): 2^26 sites, density 50, 1, 2, 3 and 4 steps
// 280 (176), 326 (352), 396 (528), 461 (704); density 100 347 (200), 439 (400),
// 557 (601); density 15 268 (174), 291 (349).  2^25 sites, 2 steps, density 50
// 151 (138), 15 124 (134), 100 201 (260).  Galilean, 2^24 sites, 3, 4 and 6 steps
// 137 (119), 164 (159), 223 (238); 2^26 sites, 2, 3 and 4 445 (361), 554 (540), 650
// (713).  C = 30, 2^24 sites, 3, 6 and 8 steps 190 (157), 327 (314), 420 (419).
void few_steps(RegWay &y, uint64_t sites, double weight, bool galilean, bool fixed) {
  constexpr double kWeight50 = 1.22;  // site_cost at density 50
  const double s = (double)sites;
  const bool cached = sites <= kCachedSites, plain = fixed && !galilean;
  y.least = 2;
  y.few_step_us = y.step_us * weight / kWeight50 * (!fixed ? 1.25 : galilean ? 1.18 : 1.0);
  y.few_launch_us = y.launch_us + (plain ? 0.0 : (cached ? 0.5e-6 : 2.0e-6) * s);
  y.few_in_us = plain && !cached ? 2.0e-6 * s : 0.0;
}
constexpr double kTileLogs = 25.0;    // the logs' records and their sum
constexpr double kStripsLaunch = 2.5;
constexpr double kUnit = 4.0;         // every further unit of a block: image and barriers
}  // namespace

std::vector<RegWay> plan_ways(const UnitPlan &plan, const uint64_t *L, uint32_t n, uint32_t blocks,
                              bool one_image, bool galilean, bool fixed, double crowded,
                              const float *cost) {
  std::vector<RegWay> ways;
  blocks = std::min(blocks, kPlanBlocks);
  uint64_t longest = 0, total = 0;
  double weight = 0;  // mean cost of a site
  bool ragged = false;
  for (uint32_t r = 0; r < n; ++r) {
    longest = std::max(longest, L[r]);
    total += L[r];
    weight += (cost ? cost[r] : 1.0) * (double)L[r];
    ragged |= L[r] % 8 != 0;
  }
  weight /= (double)total;
  for (uint32_t Q : {1u, 2u, 4u, 6u}) {
    if (!reg_has(Q, galilean, fixed, false)) continue;
    // A step's undecided sites past the queue's 64 cost every site of their
    // chunk with Q = 6: 2^24 sites, us per step with Q = 4 and 6 where 3.8 %
    // are undecided 39 and 38, 7.4 % 43 and 66, 11.5 % 45 and 73.
    if (Q == 6 && crowded > 0.1) continue;
    const bool logs = reg_has(Q, galilean, fixed, true);
    const uint64_t hold = 256ull * Q;
    if (longest <= 16 * hold) {
      RegWay y;
      y.kind = RegWay::kRing;
      y.Q = Q;
      y.most = 1u << 20;
      y.logs = logs;
      // the lattices in the order of their sizes, one per block
      double sum = 0, most = 0;
      for (uint32_t r = 0; r < n; ++r) {
        const double us = ring_step_us(Q, (uint32_t)((L[r] + hold - 1) / hold), true);
        sum += us;
        most = std::max(most, us);
      }
      const double rounds = std::max(1.0, (double)n / blocks);
      y.launch_us = kRingLaunch * rounds;
      y.step_us = std::max(most, n > blocks ? sum / blocks + 0.5 * most : 0.0);
      // (a second round of long lattices: 300 of 20000 sites, one launch of 1,
      // 2 and 3 steps 44, 64 and 84 us, and a launch per step 30, 60 and 89)
      y.least = Q == 6 && n > blocks ? 3u : 1u;
      ways.push_back(y);
      if (one_image && n > blocks && longest <= hold) {
        y.team = std::min<uint32_t>(16u, (n + blocks - 1) / blocks);
        const double r2 = std::max(1.0, (double)n / ((double)y.team * blocks));
        y.launch_us = kRingLaunch * r2;
        y.step_us = std::ceil(r2) * ring_step_us(Q, y.team, false);
        ways.push_back(y);
      }
    }
    if (plan.n_long == 0) continue;
    for (uint32_t kh : {8u, 16u, 24u, 32u, 48u, 64u, 128u}) {
      if (2 * kh >= hold) continue;
      RegWay y;
      y.kind = RegWay::kTile;
      y.Q = Q;
      y.kh = kh;
      y.most = ragged ? kh - 8 : kh;
      if (y.most == 0) continue;
      y.logs = logs && n == 1;
      const uint64_t tmax = hold - 2 * kh;
      double worst = 0, images = 0;
      for (size_t b = 0; b + 1 < plan.first.size(); ++b) {
        double us = 0;
        for (uint32_t i = plan.first[b]; i < plan.first[b + 1]; ++i) {
          const uint64_t len = plan.units[i].x1 - plan.units[i].x0;
          us += tile_step_us(Q, std::max<uint64_t>(4, (len + tmax - 1) / tmax)) *
                (cost ? cost[plan.units[i].slot] / weight : 1.0);
        }
        worst = std::max(worst, us);
        images = std::max(images, (double)(plan.first[b + 1] - plan.first[b]));
      }
      y.launch_us = kTileLaunch + (plan.strips.empty() ? 0.0 : kStripsLaunch) +
                    std::max(0.0, images - 1.0) * kUnit +
                    state_us(Q, total);
      y.step_us = worst;
      few_steps(y, total, weight, galilean, fixed);
      if (plan.n_long < n) {  // and a ring launch for the others
        y.launch_us += kRingLaunch;
        y.step_us += ring_step_us(2, 1, false) * std::max(1.0, (double)(n - plan.n_long) / blocks);
      }
      ways.push_back(y);
    }
  }
  return ways;
}

namespace {
uint64_t launches_of(const RegWay &w, uint64_t steps) {
  return w.kind == RegWay::kTile ? (steps + w.most - 1) / w.most : 1u;
}
// As the ways' estimates are compared with each other.
const RegWay *least_of(const std::vector<RegWay> &ways, uint64_t steps, bool logs, double least) {
  const RegWay *best = nullptr;
  for (const RegWay &w : ways) {
    if (logs && !w.logs) continue;
    const double us = (double)launches_of(w, steps) *
                          (w.launch_us + (logs && w.kind == RegWay::kTile ? kTileLogs : 0.0)) +
                      (double)steps * w.step_us;
    if (us < least) {
      least = us;
      best = &w;
    }
  }
  return best;
}
// As they are with other launches.
double few_us(const RegWay &w, uint64_t steps) {
  const uint64_t n = launches_of(w, steps), k = (steps + n - 1) / n;
  if (w.kind == RegWay::kRing) return w.launch_us + (double)steps * w.step_us;
  return (double)n * (w.few_launch_us + w.few_in_us / (double)k) + (double)steps * w.few_step_us;
}
}  // namespace

const RegWay *pick_way(const std::vector<RegWay> &ways, uint64_t steps, const SingleStep &single) {
  const RegWay *const best = least_of(ways, steps, false, (double)steps * single.us);
  if (!best) return nullptr;
  const uint64_t n = launches_of(*best, steps);
  if ((steps + n - 1) / n < best->least) return nullptr;
  if (best->kind == RegWay::kTile && few_us(*best, steps) >= (double)steps * single.few_us) return nullptr;
  return best;
}

// A log from the registers and one from memory, us, and what a launch of tiles
// with logs adds to one without (the kernels with logs cover little of the way
// in and out).  Measured, in launches with logs and with the moment kernels
// after each interval (every x logs): 2^27 sites 1 x 4 2740 and 1910, 2 x 8 5800
// and 6340, 3 x 1 1400 and 930, 10 x 4 8520 and 8080; 2^25 1 x 4 690 and 450, 3
// x 6 1370 and 1410; 2^24 1 x 4 307 and 274, 1 x 16 1000 and 1090, 10 x 16 4630
// and 4730; 2^22 5 x 1 84 and 71, 10 x 16 with a mode 1290 and 1580.
const RegWay *pick_log_way(const std::vector<RegWay> &ways, uint64_t every, uint64_t n_logs, uint64_t sites,
                           uint32_t n_modes, bool digest, const SingleStep &single) {
  const uint64_t steps = every * n_logs;
  const RegWay *const best = least_of(ways, steps, true, (double)steps * single.us);
  if (!best) return nullptr;
  const uint64_t n = launches_of(*best, steps), k = (steps + n - 1) / n;
  if (k < best->least) return nullptr;
  const double s = (double)sites;
  const bool large = sites > (24ull << 20);
  const RegWay *const w = pick_way(ways, every, single);
  const double apart = (w ? few_us(*w, every) + 14.0 + 0.2e-6 * s : (double)every * single.few_us) + 14.0 +
                       s * (0.9e-6 + (large ? 1.6e-6 : 0.85e-6) * n_modes + (digest ? 0.55e-6 : 0.0));
  double within = (double)n_logs * 2.0;
  if (best->kind == RegWay::kRing) {
    within += few_us(*best, steps);
  } else {
    within += (double)n * (best->few_launch_us + kTileLogs +
                           (large ? 3.6e-6 * s / (1.0 + 0.07 * (double)k) : 1.0e-6 * s / (double)k)) +
              (large ? 0.9 : 1.0) * (double)steps * best->few_step_us +
              (double)n_logs * s * ((large ? 2.6e-6 : 2.1e-6) + 1.4e-6 * n_modes + (digest ? 0.4e-6 : 0.0));
  }
  return within < (double)n_logs * apart ? best : nullptr;
}

// Measured (us per step, without and with undecided sites, 0.6 us more at 2^24
// than k_step takes since it has instances of its own for one image and fixed
// windows): 2^24 sites 37.5, 38.4 with 0.3 %, 69 with 10 %; 2^26 174, 176 and 200; of C = 30 (3 %) 52 and
// 252; 1000 lattices of 1000 sites 27, with an image each 42; 2000 of 30000 167
// and 234.
SingleStep single_step(uint64_t sites, uint32_t n, bool one_image, double missed, bool fixed) {
  const double s = (double)sites;
  SingleStep y;
  if (sites > kCachedSites) {
    y.us = 2.6e-6 * s;
    y.few_us = y.us * (fixed ? 1.0 + 1.45 * missed : 1.5) + (one_image ? 0.005 : 0.035) * n;
  } else {
    y.us = 8.0 + 2.0e-6 * s;
    y.few_us = (8.0 + 1.85e-6 * s) * (1.0 + 7.7 * missed) * (fixed ? 1.0 : 1.08) + (one_image ? 0.016 : 0.03) * n;
  }
  return y;
}

}  // namespace mclg
