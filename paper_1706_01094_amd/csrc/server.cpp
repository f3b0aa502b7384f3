// Continuous-batching server of MCLG simulation jobs.
//
// Jobs are queued on the host, admitted first-fit into a caller-owned device
// arena (their state stays resident until they finish), and advanced together
// by launches that cover the sites of all resident jobs, each job at its own
// step t (per-slot step counters on the device), several steps per launch on
// sites held in registers.  A tick is played through on the host first (which
// jobs finish when, and which queued ones take their places), then run in
// waves: wave 0 the jobs resident at its start, each for all its steps of the
// tick; wave w + 1 the jobs that took the places of wave w's finished ones.  A job's result depends only on (seed, job id, L, steps, rho, u0)
// and the collision parameters, never on what else is resident.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <deque>
#include <map>
#include <memory>
#include <new>
#include <vector>

#include "../../include/mclg.h"
#include "device.h"
#include "moments.h"
#include "regplan.h"
#include "regrun.h"
#include "tables.h"

using namespace mclg;

namespace {

constexpr uint32_t kPad = 128;
constexpr uint32_t kPoisCap = 1024;
constexpr uint32_t kImage = 160 * 1024;  // LDS collision image budget per job (at most)
constexpr size_t kImageCacheMax = 4096;   // host images kept for reuse
inline uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

struct SrvLayout {
  uint64_t o_ctrl, o_slots, o_tslot, o_tiles, o_list, o_pdesc, o_pool, o_idesc, o_over, o_ipool,
      o_rowdesc, o_thr, o_row16, bytes, max_tiles;
  // steps on sites in registers: units, their blocks, strips and their counts
  uint64_t o_units, o_ufirst, o_strips, o_sdata, o_limit;
  // moments of retiring jobs: segments, runs, partial records
  uint64_t o_mseg, o_mrun, o_mslot, o_mpart, max_mom_segs;
};

SrvLayout srv_layout(const mclg_server_config *cfg, const CollisionTables *tab,
                     uint32_t tile_sites) {
  SrvLayout l;
  uint64_t o = 0;
  auto take = [&](uint64_t b) {
    uint64_t at = o;
    o = align_up(o + b, 256);
    return at;
  };
  const uint64_t n = cfg->max_slots;
  // every resident site occupies 6 arena bytes; each slot adds one partial tile
  l.max_tiles = cfg->arena_bytes / (6ull * tile_sites) + n + 1;
  l.o_ctrl = take(256);
  l.o_slots = take(sizeof(SlotDev) * n);
  l.o_tslot = take(sizeof(uint32_t) * n);
  l.o_tiles = take(sizeof(TileDev) * l.max_tiles);
  l.o_list = take(sizeof(uint32_t) * n);
  l.max_mom_segs = max_mom_segs((uint32_t)n, cfg->arena_bytes / 6u);
  l.o_mseg = take(sizeof(MomSeg) * l.max_mom_segs);
  l.o_mrun = take(sizeof(uint32_t) * (n + 1));
  l.o_mslot = take(sizeof(uint32_t) * n);
  l.o_mpart = take(sizeof(uint64_t) * kMom3Rec * l.max_mom_segs);
  l.o_pdesc = take(sizeof(PoisDesc) * 3 * n);
  l.o_pool = take(sizeof(uint32_t) * kPoisCap * 3 * n);
  l.o_idesc = take(sizeof(ImageDesc) * n);
  l.o_over = take(kOverflowBytes);
  // (the strips' counts in the half of the overflow region that launches on
  // sites in registers leave free)
  l.o_sdata = l.o_over + kOverflowBytes / 2;
  static_assert((uint64_t)kMaxStrips * 6 * kMaxHalo * sizeof(uint16_t) <= kOverflowBytes / 2, "they fit");
  l.o_units = take(sizeof(UnitDev) * max_units((uint32_t)n));
  l.o_limit = take(sizeof(uint32_t) * n);
  l.o_ufirst = take(sizeof(uint32_t) * (kPlanBlocks + 1));
  l.o_strips = take(sizeof(StripDev) * kMaxStrips);
  l.o_ipool = take((uint64_t)kImage * n);
  l.o_rowdesc = take(sizeof(uint32_t) * tab->rowdesc.size());
  l.o_thr = take(sizeof(uint32_t) * (tab->thr.size() + 16));  // +16: see count_le_16
  l.o_row16 = take(sizeof(uint16_t) * tab->row16.size());
  l.bytes = o;
  return l;
}

struct Resident {
  mclg_job job;
  uint64_t nth = 0;     // in the order of admission
  uint64_t arena_off;   // bytes
  uint64_t bytes;
  uint64_t t = 0;
  bool active = false;
  uint32_t wave = 0, run = 0;  // its entry in the running tick's waves
};
// What a wave does with one job.
struct Run {
  uint32_t slot = 0;
  mclg_job job{};
  uint64_t nth = 0, off = 0;
  uint64_t steps = 0, t = 0;  // of the tick; the job's, when it finishes
  size_t place = 0;           // in the order of finishing
  bool fresh = false, finish = false;
};
constexpr size_t kPinned = 4u << 20;  // host memory that uploads and results go through

}  // namespace

struct mclg_server {
  mclg_server_config cfg;
  std::shared_ptr<const CollisionTables> tab;
  SrvLayout lay;
  Schedule sch;
  uint8_t *ws = nullptr;
  uint16_t *arena = nullptr;
  hipStream_t s = nullptr;
  std::deque<mclg_job> queue;
  std::vector<Resident> slot;
  std::map<uint64_t, uint64_t> free_spans;  // offset -> bytes
  uint64_t arena_used = 0;
  std::vector<mclg_job_result> done;
  std::vector<std::vector<Run>> waves;  // of the running tick
  uint32_t next_wave = 0;               // of a job admitted now
  uint64_t n_admitted = 0;
  // Pinned memory: pieces of it are handed out until it is used up, and again
  // from its start after a synchronisation.
  uint8_t *pin = nullptr;
  size_t pin_used = 0;
  Uploads pending;  // pieces to be copied before the next launch
  // finished jobs whose moments the device writes to pinned memory
  struct Finished {
    const mclg_moments_t *at;
    std::vector<std::pair<uint64_t, uint64_t>> jobs;  // (id, steps), in the moments' order
    std::vector<size_t> place;                        // in the order of finishing
  };
  std::vector<Finished> finished;
  size_t n_finished = 0;  // of the tick
  // Host images by the (rho, |u0|) they are built for: jobs of equal density
  // and speed reuse one (the image depends on u0 only through |u0|).
  struct CachedImage {
    std::vector<uint8_t> blob;
    uint32_t dir_bytes = 0, dim_a = 0, dim_c = 0, b_lo = 0, nb = 0, fixed = 0;
    double coverage = 1.0;
  };
  std::map<std::pair<double, double>, CachedImage> image_cache;
  std::vector<double> slot_coverage;  // of the image of the slot's job
  // The jobs of the last launch (their places in the order of admission) and
  // what is made of them; what of it is on the device.
  struct Planned {
    std::vector<uint64_t> jobs, sites;
    std::vector<uint32_t> list;
    uint64_t total = 0;
    UnitPlan units;
    std::vector<RegWay> ways;
    SingleStep single;
    bool list_up = false, units_up = false;
    uint32_t n_tiles = 0;  // 0: not on the device
  };
  Planned planned;
  uint32_t n_active = 0;
  uint32_t lds_bytes = 16, max_blocks = 1, image_budget = kImage, n_cu = 1;
  int last_hip = 0;

  ~mclg_server() {
    if (pin) (void)hipHostFree(pin);
  }

  uint32_t *err() { return reinterpret_cast<uint32_t *>(ws + lay.o_ctrl); }
  uint32_t *ticket() { return err() + 1; }
  SlotDev *d_slots() { return reinterpret_cast<SlotDev *>(ws + lay.o_slots); }
  uint32_t *d_tslot() { return reinterpret_cast<uint32_t *>(ws + lay.o_tslot); }
  TileDev *d_tiles() { return reinterpret_cast<TileDev *>(ws + lay.o_tiles); }
  uint32_t *d_list() { return reinterpret_cast<uint32_t *>(ws + lay.o_list); }
  uint32_t *d_limit() { return reinterpret_cast<uint32_t *>(ws + lay.o_limit); }
  TableDev table() {
    TableDev d;
    d.rowdesc = reinterpret_cast<const uint2 *>(ws + lay.o_rowdesc);
    d.thr = reinterpret_cast<const uint32_t *>(ws + lay.o_thr);
    d.row16 = tab->row16.empty() ? nullptr : reinterpret_cast<const uint4 *>(ws + lay.o_row16);
    d.row_words = tab->max_q <= 24 ? 12u : 16u;
    return d;
  }
  int hip(hipError_t e) {
    if (e == hipSuccess) return MCLG_OK;
    last_hip = (int)e;
    return MCLG_E_HIP;
  }
  hipError_t up(void *dst, const void *src, size_t bytes) {
    return bytes ? hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s) : hipSuccess;
  }

  // ---- uploads and results ------------------------------------------------
  // Waits for the device, takes the results it wrote, and frees the pinned
  // memory.
  hipError_t drain() {
    hipError_t e = hipStreamSynchronize(s);
    if (e) return e;
    for (const Finished &f : finished)
      for (size_t k = 0; k < f.jobs.size(); ++k) {
        mclg_job_result &res = done[f.place[k]];
        std::memset(&res, 0, sizeof(res));
        res.job_id = f.jobs[k].first;
        res.moments = f.at[k];
        res.moments.t = (int64_t)f.jobs[k].second;
      }
    finished.clear();
    pin_used = 0;
    return hipSuccess;
  }
  hipError_t send() {
    hipError_t e = launch_uploads(s, pending);
    pending.n = 0;
    return e;
  }
  // `bytes` (at most kPinned) of pinned memory.
  hipError_t take_pinned(size_t bytes, void *&at) {
    if (pin_used + bytes > kPinned) {
      hipError_t e = send();
      if (!e) e = drain();
      if (e) return e;
    }
    at = pin + pin_used;
    pin_used += align_up(bytes, 64);
    return hipSuccess;
  }
  // A copy of host data to the device, before the next launch after send().
  hipError_t put(void *dst, const void *src, size_t bytes) {
    for (size_t at = 0; at < bytes;) {
      const size_t n = std::min<size_t>(bytes - at, kPinned / 4);
      void *p = nullptr;
      hipError_t e = pending.n == kUploads ? send() : hipSuccess;
      if (!e) e = take_pinned(n, p);
      if (e) return e;
      std::memcpy(p, static_cast<const uint8_t *>(src) + at, n);
      pending.piece[pending.n].dst = static_cast<uint8_t *>(dst) + at;
      pending.piece[pending.n].src = p;
      pending.piece[pending.n++].bytes = n;
      at += n;
    }
    return hipSuccess;
  }
  template <class T>
  hipError_t put(void *dst, const std::vector<T> &v) { return put(dst, v.data(), sizeof(T) * v.size()); }

  bool alloc(uint64_t bytes, uint64_t &off) {
    for (auto it = free_spans.begin(); it != free_spans.end(); ++it) {
      if (it->second >= bytes) {
        off = it->first;
        uint64_t rest = it->second - bytes;
        free_spans.erase(it);
        if (rest) free_spans[off + bytes] = rest;
        arena_used += bytes;
        return true;
      }
    }
    return false;
  }
  void release(uint64_t off, uint64_t bytes) {
    arena_used -= bytes;
    auto it = free_spans.emplace(off, bytes).first;
    auto nx = std::next(it);
    if (nx != free_spans.end() && it->first + it->second == nx->first) {
      it->second += nx->second;
      free_spans.erase(nx);
    }
    if (it != free_spans.begin()) {
      auto pv = std::prev(it);
      if (pv->first + pv->second == it->first) {
        pv->second += it->second;
        free_spans.erase(it);
      }
    }
  }
  static uint64_t job_bytes(uint64_t L) { return 3 * align_up(L, kPad) * sizeof(uint16_t); }

  ImageDesc *d_idesc() { return reinterpret_cast<ImageDesc *>(ws + lay.o_idesc); }
  StepLaunch launch_args() {
    StepLaunch a{};
    a.state = arena;
    a.slots = d_slots();
    a.tslot = d_tslot();
    a.tiles = d_tiles();
    a.n_tiles = 0;
    a.slot_list = d_list();
    a.slot_first = 0;
    a.n_slots = 0;
    a.ticket = ticket();
    a.t_off = 0;
    a.single = 0;
    a.err = err();
    a.tab = table();
    a.p = params();
    a.images = d_idesc();
    a.image_pool = ws + lay.o_ipool;
    a.overflow = reinterpret_cast<uint4 *>(ws + lay.o_over);
    a.lds_bytes = lds_bytes;
    a.max_blocks = max_blocks;
    return a;
  }
  StepParams params() const {
    StepParams p;
    p.seed = cfg.seed;
    p.C = cfg.C;
    p.lam_p = cfg.lambda_num;
    p.lam_q = cfg.lambda_den;
    p.n_max = cfg.n_max;
    p.no_stream = 0;
    p.galilean = 0;
    p.tile_sites = sch.tile_sites();
    return p;
  }

  // ---- a tick on the host -------------------------------------------------
  void enter(uint32_t i, bool fresh, uint32_t wave) {
    Resident &r = slot[i];
    if (waves.size() <= wave) waves.resize(wave + 1u);
    r.wave = wave;
    r.run = (uint32_t)waves[wave].size();
    Run x;
    x.slot = i;
    x.job = r.job;
    x.nth = r.nth;
    x.off = r.arena_off;
    x.fresh = fresh;
    waves[wave].push_back(x);
  }
  // Admit queued jobs (FIFO, stop at the first that does not fit).
  void admit() {
    while (!queue.empty()) {
      const mclg_job &j = queue.front();
      uint32_t free_slot = UINT32_MAX;
      for (uint32_t i = 0; i < slot.size(); ++i)
        if (!slot[i].active) { free_slot = i; break; }
      if (free_slot == UINT32_MAX) break;
      uint64_t bytes = job_bytes(j.L), off = 0;
      if (!alloc(bytes, off)) break;
      Resident &r = slot[free_slot];
      r.job = j;
      r.nth = n_admitted++;
      r.arena_off = off;
      r.bytes = bytes;
      r.t = 0;
      r.active = true;
      ++n_active;
      enter(free_slot, true, next_wave);
      queue.pop_front();
    }
  }
  void advance(uint64_t k) {
    for (auto &r : slot)
      if (r.active) {
        r.t += k;
        waves[r.wave][r.run].steps += k;
      }
  }
  // Free the slots of finished jobs.  What is admitted from here on may take
  // their places, so it runs after them.
  void retire() {
    for (auto &r : slot)
      if (r.active && r.t >= r.job.steps) {
        Run &x = waves[r.wave][r.run];
        x.finish = true;
        x.t = r.t;
        x.place = n_finished++;
        next_wave = std::max(next_wave, r.wave + 1u);
        r.active = false;
        --n_active;
        release(r.arena_off, r.bytes);
      }
  }

  // ---- a wave on the device -----------------------------------------------
  hipError_t start_jobs(const std::vector<Run> &wave) {
    std::vector<uint32_t> fresh, pool;
    std::vector<TileDev> tiles;
    const uint32_t ts = sch.tile_sites();
    hipError_t e = hipSuccess;
    for (const Run &r : wave) {
      if (!r.fresh) continue;
      SlotDev sd{};
      sd.off = r.off / sizeof(uint16_t);
      sd.dense = 0;
      sd.L = (uint32_t)r.job.L;
      sd.stride = (uint32_t)align_up(r.job.L, kPad);
      sd.rid = (uint32_t)r.job.job_id;
      sd.pad = 0;
      double mu[3];
      feq(r.job.rho, r.job.u0, mu);
      PoisDesc pd[3];
      for (int i = 0; i < 3; ++i) {
        uint32_t k_lo = 0;
        std::vector<uint64_t> full;
        poisson_full(mu[i], k_lo, full);
        CompactLaw cl = compact(k_lo, full);
        pd[i].off = (uint32_t)pool.size();
        pd[i].k_first = cl.k_first;
        pd[i].nthr = (uint32_t)cl.thr.size();
        pool.insert(pool.end(), cl.thr.begin(), cl.thr.end());
      }
      // collision image for this job's density and speed (cached on the host)
      const auto key = std::make_pair(r.job.rho, std::fabs(r.job.u0));
      auto ci = image_cache.find(key);
      if (ci == image_cache.end()) {
        if (image_cache.size() >= kImageCacheMax) image_cache.clear();
        LdsImage im = build_image(*tab, r.job.rho, std::fabs(r.job.u0), image_budget);
        CachedImage c;
        c.blob = im.blob();
        c.dir_bytes = im.dir_bytes();
        c.dim_a = im.dim_a;
        c.dim_c = im.dim_c;
        c.b_lo = im.b_lo;
        c.nb = im.nb;
        c.fixed = im.fixed ? 1u : 0u;
        c.coverage = im.coverage;
        ci = image_cache.emplace(key, std::move(c)).first;
      }
      const CachedImage &img = ci->second;
      slot_coverage[r.slot] = img.coverage;
      ImageDesc idd{};
      idd.off = (uint64_t)r.slot * kImage;
      idd.bytes = (uint32_t)img.blob.size();
      idd.dir_bytes = img.dir_bytes;
      idd.dim_a = img.dim_a;
      idd.dim_c = img.dim_c;
      idd.b_lo = img.b_lo;
      idd.nb = img.nb;
      idd.fixed = img.fixed;
      idd.skew = image_skew(img.coverage);
      if (!e) e = put(ws + lay.o_ipool + idd.off, img.blob);
      if (!e) e = put(d_slots() + r.slot, &sd, sizeof(sd));
      if (!e) e = put(d_idesc() + r.slot, &idd, sizeof(idd));
      if (!e) e = put(ws + lay.o_pdesc + sizeof(PoisDesc) * 3 * r.slot, pd, sizeof(pd));
      fresh.push_back(r.slot);
      for (uint64_t x0 = 0; x0 < r.job.L; x0 += ts) tiles.push_back(TileDev{r.slot, (uint32_t)x0, 0, 0});
    }
    if (fresh.empty() || e) return e;
    if (tiles.size() > lay.max_tiles) return hipErrorInvalidValue;
    planned.list_up = false;
    planned.n_tiles = 0;
    e = put(ws + lay.o_pool, pool);
    if (!e) e = put(d_list(), fresh);
    if (!e) e = put(d_tiles(), tiles);
    if (!e) e = send();
    if (!e) e = launch_set_t(s, d_tslot(), d_list(), (uint32_t)fresh.size(), 0u);
    if (!e)
      e = launch_init_poisson(s, arena, d_slots(), d_tslot(), d_tiles(), (uint32_t)tiles.size(), ts,
                              reinterpret_cast<const PoisDesc *>(ws + lay.o_pdesc),
                              reinterpret_cast<const uint32_t *>(ws + lay.o_pool), cfg.seed, err());
    return e;
  }

  // The lists that launches read, for the jobs of `left` that have steps left:
  // made anew only when those are others than the last ones, and uploaded only
  // when the device holds others (a tick of few steps is no longer than its
  // uploads).
  hipError_t plan_jobs(const std::vector<Run> &wave, const std::vector<uint64_t> &left, size_t n) {
    Planned &p = planned;
    bool same = p.jobs.size() == n;
    for (size_t i = 0, k = 0; same && i < wave.size(); ++i)
      if (left[i]) same = p.jobs[k++] == wave[i].nth;
    if (same) return hipSuccess;
    p = Planned();
    uint64_t crowd = 0;
    double missed = 0;
    std::vector<float> cost;
    for (size_t i = 0; i < wave.size(); ++i)
      if (left[i]) {
        const double cov = slot_coverage[wave[i].slot];
        missed += cfg.C ? (1.0 - cov) * (double)wave[i].job.L : 0.0;
        crowd += crowded_image(cov) ? wave[i].job.L : 0u;
        cost.push_back(cfg.C ? site_cost(cov) : 1.0f);
        p.jobs.push_back(wave[i].nth);
        p.list.push_back(wave[i].slot);
        p.sites.push_back(wave[i].job.L);
        p.total += wave[i].job.L;
      }
    p.units = plan_units(p.sites.data(), (uint32_t)n, n_cu, cost.data());
    if (p.units.units.size() > max_units((uint32_t)slot.size())) {
      p = Planned();
      return hipErrorInvalidValue;
    }
    p.ways = plan_ways(p.units, p.sites.data(), (uint32_t)n, n_cu, false, false, images_fixed(cfg.C),
                       (double)crowd / (double)p.total, cost.data());
    p.single = single_step(p.total, (uint32_t)n, n == 1, missed / (double)p.total, images_fixed(cfg.C));
    for (UnitDev &u : p.units.units) u.slot = p.list[u.slot];
    for (StripDev &x : p.units.strips) x.slot = p.list[x.slot];
    return hipSuccess;
  }

  // The steps of a wave's jobs: launches that each job takes part in for as
  // many steps as it has left.
  hipError_t step_jobs(std::vector<Run> &wave) {
    std::stable_sort(wave.begin(), wave.end(), [](const Run &x, const Run &y) { return x.job.L > y.job.L; });
    std::vector<uint64_t> left(wave.size());
    for (size_t i = 0; i < wave.size(); ++i) left[i] = wave[i].steps;
    for (;;) {
      uint64_t most = 0, least = ~0ull;
      size_t n = 0;
      for (uint64_t k : left)
        if (k) {
          most = std::max(most, k);
          least = std::min(least, k);
          ++n;
        }
      if (n == 0) return hipSuccess;
      hipError_t e = plan_jobs(wave, left, n);
      if (e) return e;
      Planned &p = planned;
      StepLaunch a = launch_args();
      a.n_slots = (uint32_t)n;
      if (!p.list_up) e = put(d_list(), p.list);
      const RegWay *w = pick_way(p.ways, most, p.single);
      uint64_t m = least;  // the launch's steps
      if (!w) {
        const uint32_t ts = sch.tile_sites();
        if (!p.n_tiles) {
          std::vector<TileDev> tiles;
          for (size_t i = 0; i < n; ++i) {
            const uint32_t next = (uint32_t)(tiles.size() + (p.sites[i] + ts - 1) / ts);
            for (uint64_t x0 = 0; x0 < p.sites[i]; x0 += ts) tiles.push_back(TileDev{p.list[i], (uint32_t)x0, next, 0});
          }
          if (tiles.size() > lay.max_tiles) e = hipErrorInvalidValue;
          if (!e) e = put(d_tiles(), tiles);
          if (!e) p.n_tiles = (uint32_t)tiles.size();
        }
        a.n_tiles = p.n_tiles;
        a.p.drain = auto_drain(6 * p.total);  // by the jobs' state
        if (!e) e = send();
        if (!e) p.list_up = true;
        for (uint64_t i = 0; i < m && !e; ++i) e = launch_step(sch, s, a);
      } else {
        const uint64_t launches = (most + w->most - 1) / w->most;
        m = (most + launches - 1) / launches;
        // alone on the device, and all of them for as many steps: no limits
        const bool all = waves.size() == 1 && n == wave.size() && least >= m;
        if (!all) {
          std::vector<uint32_t> limit(slot.size(), 0u);
          for (size_t i = 0; i < wave.size(); ++i) limit[wave[i].slot] = (uint32_t)std::min(left[i], m);
          if (!e) e = put(d_limit(), limit);
        }
        if (!p.units_up) {
          if (!e) e = put(ws + lay.o_units, p.units.units);
          if (!e) e = put(ws + lay.o_ufirst, p.units.first);
          if (!e) e = put(ws + lay.o_strips, p.units.strips);
        }
        if (!e) e = send();
        if (!e) p.list_up = p.units_up = true;
        RegBufs b;
        b.order = d_list();
        b.n = (uint32_t)n;
        b.units = reinterpret_cast<const UnitDev *>(ws + lay.o_units);
        b.first = reinterpret_cast<const uint32_t *>(ws + lay.o_ufirst);
        b.strips = reinterpret_cast<const StripDev *>(ws + lay.o_strips);
        b.strip_data = reinterpret_cast<uint16_t *>(ws + lay.o_sdata);
        b.limit = all ? nullptr : d_limit();
        if (!e) e = launch_way(s, a, *w, p.units, b, (uint32_t)m, RegLog());
        // (a free slot's counter is set when a job takes it)
        if (!e)
          e = all ? launch_add_t(s, d_tslot(), 0, (uint32_t)slot.size(), (uint32_t)m)
                  : launch_add_each(s, d_tslot(), d_limit(), (uint32_t)slot.size());
      }
      if (e) return e;
      for (uint64_t &k : left) k -= std::min(k, m);
    }
  }

  // Moments (with the state digest) of a wave's finished jobs.
  hipError_t finish_jobs(const std::vector<Run> &wave) {
    std::vector<uint32_t> fin;
    std::vector<uint64_t> sites;
    Finished f;
    for (const Run &r : wave)
      if (r.finish) {
        fin.push_back(r.slot);
        sites.push_back(r.job.L);
        f.jobs.emplace_back(r.job.job_id, r.t);
        f.place.push_back(r.place);
      }
    // (a slot is in a wave once, and its results fit the pinned memory)
    const size_t most = kPinned / 4 / sizeof(mclg_moments_t);
    for (size_t i0 = 0; i0 < fin.size(); i0 += most) {
      const uint32_t n = (uint32_t)std::min(most, fin.size() - i0);
      const MomPlan plan = plan_moments(fin.data() + i0, sites.data() + i0, n);
      if (plan.segs.size() > lay.max_mom_segs) return hipErrorInvalidValue;
      MomArgs m;
      m.state = arena;
      m.slots = d_slots();
      m.tslot = d_tslot();
      m.segs = reinterpret_cast<const MomSeg *>(ws + lay.o_mseg);
      m.n_segs = (uint32_t)plan.segs.size();
      m.run_seg = reinterpret_cast<const uint32_t *>(ws + lay.o_mrun);
      m.run_slot = reinterpret_cast<const uint32_t *>(ws + lay.o_mslot);
      m.n_runs = n;
      m.digest = 1u;
      m.partial = reinterpret_cast<unsigned long long *>(ws + lay.o_mpart);
      hipError_t e = put(ws + lay.o_mseg, plan.segs);
      if (!e) e = put(ws + lay.o_mrun, plan.run_seg);
      if (!e) e = put(ws + lay.o_mslot, plan.run_slot);
      void *at = nullptr;
      if (!e) e = take_pinned(sizeof(mclg_moments_t) * n, at);
      if (!e) e = send();
      m.out = static_cast<long long *>(at);
      if (!e) e = launch_moments3(s, m);
      if (e) return e;
      Finished part;
      part.at = static_cast<const mclg_moments_t *>(at);
      part.jobs.assign(f.jobs.begin() + i0, f.jobs.begin() + i0 + n);
      part.place.assign(f.place.begin() + i0, f.place.begin() + i0 + n);
      finished.push_back(std::move(part));
    }
    return hipSuccess;
  }

  // After an error the host's account of the tick is not the device's state:
  // its jobs, finished ones too, go back to the head of the queue in the order
  // of their admission, and run anew when they are admitted again.
  void start_over() {
    std::vector<const Run *> runs;
    for (const auto &wave : waves)
      for (const Run &r : wave) runs.push_back(&r);
    std::sort(runs.begin(), runs.end(), [](const Run *x, const Run *y) { return x->nth > y->nth; });
    for (const Run *r : runs) queue.push_front(r->job);
    for (Resident &r : slot) r.active = false;
    n_active = 0;
    free_spans.clear();
    if (const uint64_t usable = cfg.arena_bytes / 256 * 256) free_spans[0] = usable;
    arena_used = 0;
    planned = Planned();
    pending.n = 0;
    if (!hipStreamSynchronize(s)) pin_used = 0;
  }

  // What the tick did on the host, on the device.
  hipError_t run_waves() {
    const size_t before = done.size();
    done.resize(before + n_finished);
    hipError_t e = hipSuccess;
    for (auto &wave : waves) {
      for (Run &r : wave) r.place += before;
      if (!e) e = start_jobs(wave);
      if (!e) e = step_jobs(wave);
      if (!e) e = finish_jobs(wave);
    }
    if (!e && !finished.empty()) e = drain();
    if (e) {  // no results of this tick
      finished.clear();
      done.resize(before);
      start_over();
    }
    return e;
  }
};

extern "C" {

int mclg_server_sizes(const mclg_server_config *cfg, uint64_t *workspace_bytes) {
  if (!cfg || cfg->abi_version != MCLG_ABI_VERSION || cfg->max_slots == 0 || !workspace_bytes)
    return MCLG_E_INVAL;
  if (!params_ok(cfg->C, cfg->lambda_num, cfg->lambda_den, cfg->n_max, false))
    return MCLG_E_INVAL;
  auto tab = collision_tables(cfg->C, cfg->lambda_num, cfg->lambda_den, cfg->n_max, false);
  if (!tab) return MCLG_E_INVAL;
  Schedule sch;
  *workspace_bytes = srv_layout(cfg, tab.get(), sch.tile_sites()).bytes;
  return MCLG_OK;
}

int mclg_server_create(const mclg_server_config *cfg, mclg_server **out) {
  uint64_t need = 0;
  int rc = mclg_server_sizes(cfg, &need);
  if (rc) return rc;
  if (!out || !cfg->arena || !cfg->workspace || cfg->workspace_bytes < need) return MCLG_E_INVAL;
  std::unique_ptr<mclg_server> sv(new (std::nothrow) mclg_server());
  if (!sv) return MCLG_E_NOMEM;
  sv->cfg = *cfg;
  sv->tab = collision_tables(cfg->C, cfg->lambda_num, cfg->lambda_den, cfg->n_max, false);
  sv->lay = srv_layout(cfg, sv->tab.get(), sv->sch.tile_sites());
  sv->ws = reinterpret_cast<uint8_t *>(cfg->workspace);
  sv->arena = reinterpret_cast<uint16_t *>(cfg->arena);
  sv->s = reinterpret_cast<hipStream_t>(cfg->stream);
  sv->slot.resize(cfg->max_slots);
  sv->slot_coverage.assign(cfg->max_slots, 1.0);
  {
    int dev = 0, v = 0;
    hipError_t e = hipGetDevice(&dev);
    if (!e) e = hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    const uint32_t queues = (sv->sch.threads / 64u) * kWaveLdsBytes;
    if (!e) sv->image_budget = std::min<uint32_t>(kImage, (uint32_t)std::max(0, v - 1024 - (int)queues)) / 16u * 16u;
    if (!e) e = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev);
    if (!e) sv->n_cu = (uint32_t)std::max(1, v);
    if (!e && sv->n_cu > 256) return MCLG_E_UNSUPPORTED;  // overflow region sized for 256 CUs
    sv->lds_bytes = std::max<uint32_t>(64, sv->image_budget);  // the smallest image is 48 bytes
    if (!e) e = reg_setup(sv->lds_bytes);
    if (!e) e = step_occupancy(sv->sch, sv->lds_bytes, sv->n_cu, sv->max_blocks);
    if (e) return sv->hip(e);
  }
  uint64_t usable = cfg->arena_bytes / 256 * 256;
  if (usable) sv->free_spans[0] = usable;
  {
    hipError_t e = hipHostMalloc(reinterpret_cast<void **>(&sv->pin), kPinned, hipHostMallocDefault);
    if (e) return sv->hip(e);
  }
  std::vector<uint32_t> ctrl(64, 0), tz(cfg->max_slots, 0);
  const CollisionTables &t = *sv->tab;
  hipError_t e = sv->up(sv->ws + sv->lay.o_ctrl, ctrl.data(), 256);
  if (!e) e = sv->up(sv->d_tslot(), tz.data(), 4 * tz.size());
  if (!e) e = sv->up(sv->ws + sv->lay.o_rowdesc, t.rowdesc.data(), 4 * t.rowdesc.size());
  if (!e) e = sv->up(sv->ws + sv->lay.o_thr, t.thr.data(), 4 * t.thr.size());
  if (!e && !t.row16.empty()) e = sv->up(sv->ws + sv->lay.o_row16, t.row16.data(), 2 * t.row16.size());
  if (!e) e = hipStreamSynchronize(sv->s);
  if (e) return sv->hip(e);
  *out = sv.release();
  return MCLG_OK;
}

int mclg_server_submit(mclg_server *sv, const mclg_job *job) {
  if (!sv || !job || job->L == 0 || job->L > kMaxSites || job->job_id >= (1ull << 32))
    return MCLG_E_INVAL;
  if (!(job->rho >= 0.0) || !(job->u0 >= -1.0 && job->u0 <= 1.0)) return MCLG_E_INVAL;
  if (mclg_server::job_bytes(job->L) > sv->cfg.arena_bytes / 256 * 256) return MCLG_E_INVAL;
  double mu[3];
  feq(job->rho, job->u0, mu);
  for (double m : mu) {
    uint32_t k_lo = 0;
    std::vector<uint64_t> full;
    if (!poisson_full(m, k_lo, full) || compact(k_lo, full).thr.size() > kPoisCap) return MCLG_E_INVAL;
  }
  sv->queue.push_back(*job);
  return MCLG_OK;
}

int mclg_server_tick(mclg_server *sv, uint32_t k) {
  if (!sv) return MCLG_E_INVAL;
  sv->waves.clear();
  sv->next_wave = 0;
  sv->n_finished = 0;
  for (uint32_t i = 0; i < sv->slot.size(); ++i)
    if (sv->slot[i].active) sv->enter(i, false, 0);
  sv->admit();
  for (uint32_t left = k; left > 0 && sv->n_active > 0;) {
    uint64_t chunk = left;
    for (auto &r : sv->slot)
      if (r.active) chunk = std::min<uint64_t>(chunk, r.job.steps - r.t);
    sv->advance(chunk);
    left -= (uint32_t)chunk;
    sv->retire();
    sv->admit();
  }
  return sv->hip(sv->run_waves());
}

int mclg_server_poll(mclg_server *sv, mclg_job_result *out, uint32_t cap, uint32_t *n_out) {
  if (!sv || !n_out || (cap && !out)) return MCLG_E_INVAL;
  uint32_t n = (uint32_t)std::min<size_t>(cap, sv->done.size());
  std::copy(sv->done.begin(), sv->done.begin() + n, out);
  sv->done.erase(sv->done.begin(), sv->done.begin() + n);
  *n_out = n;
  uint32_t err = 0;
  hipError_t e = hipMemcpy(&err, sv->err(), sizeof(err), hipMemcpyDeviceToHost);
  if (e) return sv->hip(e);
  return err ? MCLG_E_RANGE : MCLG_OK;
}

int mclg_server_stats(const mclg_server *sv, uint64_t *queued, uint64_t *resident,
                      uint64_t *arena_used) {
  if (!sv) return MCLG_E_INVAL;
  if (queued) *queued = sv->queue.size();
  if (resident) *resident = sv->n_active;
  if (arena_used) *arena_used = sv->arena_used;
  return MCLG_OK;
}

int mclg_server_destroy(mclg_server *sv) {
  if (!sv) return MCLG_E_INVAL;
  // (on the null stream too: a tick may have left launches that read the pinned
  // memory)
  (void)hipStreamSynchronize(sv->s);
  delete sv;
  return MCLG_OK;
}

}  // extern "C"
