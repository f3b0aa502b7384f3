"""The server's host side over a device that fails (host side, compiled here;
the HIP calls and the kernels are stand-ins that work on host memory, one of
which returns an error): a failed tick loses no job, the pinned memory that
the device reads is never freed before the device is done with it, and a tick
with the same jobs as the last one uploads nothing."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(__file__))
CSRC = os.path.join(ROOT, "paper_1706_01094_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include "device.h"
#include "moments.h"
#include "regplan.h"
#include "../../include/mclg.h"
using namespace mclg;
static bool busy = false, freed_busy = false;
static size_t uploads = 0;
static long calls = 0, fail_at = 0;  // the fail_at-th call from now on fails
static hipError_t call() { return fail_at && ++calls == fail_at ? hipErrorOutOfMemory : hipSuccess; }
extern "C" {
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  hipError_t e = call();
  if (!e) std::memcpy(d, s, n);
  return e;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { busy = false; return call(); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { freed_busy |= busy; std::free(p); return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024;
  return hipSuccess;
}
}
static hipError_t launch() { hipError_t e = call(); busy |= !e; return e; }
static std::map<const void *, uint64_t> start;  // of a job's state: its id
namespace mclg {
bool reg_has(uint32_t Q, bool g, bool f, bool l) { return l ? !g && f && Q <= 4 : f ? !g || Q <= 2 : Q == 2; }
hipError_t reg_setup(uint32_t) { return hipSuccess; }
hipError_t step_occupancy(const Schedule &, uint32_t, uint32_t n, uint32_t &b) { b = n; return hipSuccess; }
hipError_t launch_ring(hipStream_t, const StepLaunch &, const RingLaunch &, uint32_t, uint32_t) { return launch(); }
hipError_t launch_tiles(hipStream_t, const StepLaunch &, const TileLaunch &, uint32_t, uint32_t, uint32_t, const uint32_t *) {
  return launch();
}
hipError_t launch_step(const Schedule &, hipStream_t, const StepLaunch &a) {
  hipError_t e = launch();
  for (uint32_t k = 0; !e && k < a.n_slots; ++k) ++a.tslot[a.slot_list[k]];
  return e;
}
hipError_t launch_uploads(hipStream_t, const Uploads &u) {
  if (!u.n) return hipSuccess;
  uploads += u.n;
  hipError_t e = launch();
  for (uint32_t k = 0; !e && k < u.n; ++k) std::memcpy(u.piece[k].dst, u.piece[k].src, u.piece[k].bytes);
  return e;
}
hipError_t launch_set_t(hipStream_t, uint32_t *t, const uint32_t *list, uint32_t n, uint32_t v) {
  hipError_t e = launch();
  for (uint32_t k = 0; !e && k < n; ++k) t[list[k]] = v;
  return e;
}
hipError_t launch_add_t(hipStream_t, uint32_t *t, uint32_t first, uint32_t n, uint32_t add) {
  hipError_t e = launch();
  for (uint32_t k = 0; !e && k < n; ++k) t[first + k] += add;
  return e;
}
hipError_t launch_add_each(hipStream_t, uint32_t *t, const uint32_t *add, uint32_t n) {
  hipError_t e = launch();
  for (uint32_t k = 0; !e && k < n; ++k) t[k] += add[k];
  return e;
}
hipError_t launch_init_poisson(hipStream_t, uint16_t *state, const SlotDev *s, const uint32_t *, const TileDev *tiles,
                               uint32_t n, uint32_t, const PoisDesc *, const uint32_t *, uint64_t, uint32_t *) {
  hipError_t e = launch();
  for (uint32_t k = 0; !e && k < n; ++k) start[state + s[tiles[k].slot].off] = s[tiles[k].slot].rid;
  return e;
}
hipError_t launch_moments3(hipStream_t, const MomArgs &a) {
  hipError_t e = launch();
  for (uint32_t j = 0; !e && j < a.n_runs; ++j) {
    const SlotDev &s = a.slots[a.run_slot[j]];
    long long *o = a.out + (uint64_t)j * kMom3Out;
    std::memset(o, 0, 8 * kMom3Out);
    o[0] = a.tslot[a.run_slot[j]];
    o[1] = s.L;
    o[2] = (long long)start[a.state + s.off];
  }
  return e;
}
MomPlan plan_moments(const uint32_t *slots, const uint64_t *sites, uint32_t n) {
  MomPlan p;
  p.run_seg.push_back(0);
  for (uint32_t j = 0; j < n; ++j) {
    MomSeg m;
    m.slot = slots[j]; m.x1 = (uint32_t)sites[j]; m.run = j;
    p.segs.push_back(m);
    p.run_seg.push_back(j + 1);
    p.run_slot.push_back(slots[j]);
  }
  return p;
}
}
#define REQUIRE(x) if (!(x)) { std::printf("tick %u, call %ld: %s\n", tick, at, #x); std::exit(1); }
static int ticks() {
  const uint32_t n = 14;
  for (uint32_t tick : {3u, 8u, 60u}) {
    long last = 1;
    for (long at = 0; at <= last; ++at) {  // 0: no failure
      mclg_server_config c{};
      c.abi_version = MCLG_ABI_VERSION;
      c.max_slots = 4;
      c.seed = 1;
      c.C = 2;
      c.lambda_num = c.lambda_den = 1;
      c.n_max = 40;
      c.arena_bytes = 60000;
      uint64_t need = 0;
      calls = fail_at = 0;
      REQUIRE(mclg_server_sizes(&c, &need) == MCLG_OK);
      c.arena = std::malloc(c.arena_bytes);
      c.workspace = std::malloc(need);
      c.workspace_bytes = need;
      mclg_server *sv = nullptr;
      REQUIRE(mclg_server_create(&c, &sv) == MCLG_OK);
      auto job = [&](uint32_t i) {
        return mclg_job{i, 1 + 977ull * i % 3000, (uint64_t)(7 * i % 20), 5.0 + i % 3, 0.0};
      };
      for (uint32_t i = 0; i < n; ++i) {
        const mclg_job j = job(i);
        REQUIRE(mclg_server_submit(sv, &j) == MCLG_OK);
      }
      calls = 0;
      fail_at = at ? at : 1l << 40;
      std::map<uint64_t, mclg_moments_t> got;
      int failed = 0;
      for (int k = 0; k < 400 && got.size() < n; ++k) {
        const int rc = mclg_server_tick(sv, tick);
        REQUIRE(rc == MCLG_OK || (rc == MCLG_E_HIP && at && !failed));
        failed += rc != MCLG_OK;
        mclg_job_result r[3];
        uint32_t m = 0;
        do {
          REQUIRE(mclg_server_poll(sv, r, 3, &m) == MCLG_OK);
          for (uint32_t i = 0; i < m; ++i) REQUIRE(got.emplace(r[i].job_id, r[i].moments).second);
        } while (m);
      }
      if (!at) last = calls;
      REQUIRE(failed == (at ? 1 : 0));
      uint64_t queued = 1, resident = 1, used = 1;
      REQUIRE(mclg_server_stats(sv, &queued, &resident, &used) == MCLG_OK && !queued && !resident && !used);
      REQUIRE(got.size() == n);
      for (uint32_t i = 0; i < n; ++i) {
        const mclg_job j = job(i);
        REQUIRE(got.count(i) && got[i].t == (int64_t)j.steps && got[i].sites == (int64_t)j.L && got[i].sum_n[0] == i);
      }
      mclg_server_destroy(sv);
      REQUIRE(!freed_busy);
      std::free(c.arena);
      std::free(c.workspace);
    }
    REQUIRE_LAST
  }
  return 0;
}
// Left with work in flight on the null stream.
static int end() {
  mclg_server_config c{};
  c.abi_version = MCLG_ABI_VERSION;
  c.max_slots = 1;
  c.C = 2;
  c.lambda_num = c.lambda_den = 1;
  c.n_max = 40;
  c.arena_bytes = 60000;
  uint64_t need = 0;
  fail_at = 0;
  busy = freed_busy = false;
  uint32_t tick = 0;
  long at = 0;
  REQUIRE(mclg_server_sizes(&c, &need) == MCLG_OK);
  c.arena = std::malloc(c.arena_bytes);
  c.workspace = std::malloc(need);
  c.workspace_bytes = need;
  mclg_server *sv = nullptr;
  const mclg_job j{0, 1000, 50, 5.0, 0.0};
  REQUIRE(mclg_server_create(&c, &sv) == MCLG_OK && mclg_server_submit(sv, &j) == MCLG_OK && mclg_server_tick(sv, 3) == MCLG_OK);
  REQUIRE(busy);
  mclg_server_destroy(sv);
  REQUIRE(!freed_busy);
  return 0;
}
// Ticks of any length between jobs that join.
static int steady() {
  mclg_server_config c{};
  c.abi_version = MCLG_ABI_VERSION;
  c.max_slots = 9;
  c.C = 2;
  c.lambda_num = c.lambda_den = 1;
  c.n_max = 40;
  c.arena_bytes = 900000;
  uint64_t need = 0;
  fail_at = 0;
  uint32_t tick = 0;
  long at = 0;
  REQUIRE(mclg_server_sizes(&c, &need) == MCLG_OK);
  c.arena = std::malloc(c.arena_bytes);
  c.workspace = std::malloc(need);
  c.workspace_bytes = need;
  mclg_server *sv = nullptr;
  REQUIRE(mclg_server_create(&c, &sv) == MCLG_OK);
  for (uint32_t i = 0; i < 4; ++i) {
    const mclg_job j{i, 500 + 9000ull * i, 100000, 5.0, 0.0};
    REQUIRE(mclg_server_submit(sv, &j) == MCLG_OK);
    const uint32_t lengths[] = {1, 40, 2, 300};
    for (int round = 0; round < 3; ++round)
      for (uint32_t k : lengths) {
        tick = k;
        uploads = 0;
        REQUIRE(mclg_server_tick(sv, k) == MCLG_OK);
        REQUIRE(round == 0 || uploads == 0);
      }
  }
  REQUIRE(mclg_server_destroy(sv) == MCLG_OK);
  return 0;
}
int main(int argc, char **argv) {
  if (argc < 2 ? ticks() : argv[1][0] == 'e' ? end() : steady()) return 1;
  std::puts("ok");
}
"""
MAIN = MAIN.replace("    REQUIRE_LAST\n", "")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("server")
    src, exe = tmp / "main.cpp", tmp / "main"
    src.write_text(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-o", str(exe), str(src)] + [os.path.join(CSRC, f) for f in ("server.cpp", "regplan.cpp", "tables.cpp")],
                   check=True)
    return str(exe)


@pytest.mark.parametrize("args", [[], ["end"], ["steady"]], ids=["ticks", "end", "steady"])
def test_server_over_a_failing_device(program, args):
    out = subprocess.run([program] + args, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
