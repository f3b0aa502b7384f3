"""Contexts where the host has no pinned memory to give (host side, compiled
here; the HIP calls and the kernels are stand-ins that work on host memory):
accepted, and their moments read through a copy."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(__file__))
CSRC = os.path.join(ROOT, "paper_1706_01094_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "d2q9.h"
#include "device.h"
#include "moments.h"
#include "../../include/mclg.h"
using namespace mclg;
static bool none = false;        // no pinned memory
static hipError_t last = hipSuccess;  // the runtime's, until it is read
extern "C" {
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  if (none) return last = hipErrorOutOfMemory;
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipGetLastError() { hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
}
namespace mclg {
static unsigned long long area[16];
hipError_t moments_scratch(unsigned long long **p) { *p = area; return hipGetLastError(); }
bool reg_has(uint32_t, bool, bool, bool) { return false; }
hipError_t reg_setup(uint32_t) { return hipGetLastError(); }
hipError_t step_occupancy(const Schedule &, uint32_t, uint32_t n, uint32_t &b) { b = n; return hipGetLastError(); }
hipError_t launch_ring(hipStream_t, const StepLaunch &, const RingLaunch &, uint32_t, uint32_t) { return hipGetLastError(); }
hipError_t launch_tiles(hipStream_t, const StepLaunch &, const TileLaunch &, uint32_t, uint32_t, uint32_t, const uint32_t *) {
  return hipGetLastError();
}
hipError_t launch_step(const Schedule &, hipStream_t, const StepLaunch &) { return hipGetLastError(); }
hipError_t launch_init_poisson(hipStream_t, uint16_t *, const SlotDev *, const uint32_t *, const TileDev *, uint32_t, uint32_t,
                               const PoisDesc *, const uint32_t *, uint64_t, uint32_t *) { return hipGetLastError(); }
hipError_t launch_init_counts(hipStream_t, uint16_t *, const SlotDev *, const TileDev *, uint32_t, uint32_t, const uint16_t *) {
  return hipGetLastError();
}
hipError_t launch_histogram(hipStream_t, const uint16_t *, const SlotDev *, const TileDev *, uint32_t, uint32_t, uint32_t,
                            unsigned long long *) { return hipGetLastError(); }
hipError_t launch_add_t(hipStream_t, uint32_t *t, uint32_t first, uint32_t n, uint32_t add) {
  for (uint32_t k = 0; k < n; ++k) t[first + k] += add;
  return hipGetLastError();
}
hipError_t launch_step9(hipStream_t, const Step9 &, uint32_t) { return hipGetLastError(); }
hipError_t launch_steps9(hipStream_t, const Step9 &, uint32_t, uint32_t, uint32_t) { return hipGetLastError(); }
hipError_t launch_init9_poisson(hipStream_t, uint16_t *, const Rep9 *, const Tile9 *, uint32_t, const PoisDesc *, const uint32_t *,
                                uint64_t, uint32_t *) { return hipGetLastError(); }
hipError_t launch_init9_counts(hipStream_t, uint16_t *, const Rep9 *, const Tile9 *, uint32_t, const uint64_t *, const uint16_t *,
                               uint32_t *) { return hipGetLastError(); }
hipError_t launch_histogram9(hipStream_t, const uint16_t *, const Rep9 *, const Tile9 *, uint32_t, uint32_t, unsigned long long *) {
  return hipGetLastError();
}
static hipError_t moments(const MomArgs &a, uint32_t words) {
  for (uint32_t j = 0; j < a.n_runs; ++j) {
    long long *o = a.out + (uint64_t)j * words;
    std::memset(o, 0, 8 * words);
    o[1] = 7 + j;
  }
  if (a.err) a.out[(uint64_t)a.n_runs * words] = *a.err;
  return hipGetLastError();
}
hipError_t launch_moments3(hipStream_t, const MomArgs &a) { return moments(a, kMom3Out); }
hipError_t launch_moments9(hipStream_t, const MomArgs &a) { return moments(a, kMom9Out); }
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
#define REQUIRE(x) if (!(x)) { std::printf("%d %d: %s\n", lattice, (int)none, #x); return 1; }
int main() {
  const uint64_t L[2] = {40, 9}, Ly[2] = {3, 5};
  uint32_t lam[18];
  for (int i = 0; i < 18; ++i) lam[i] = i & 1 ? 8 : 1;
  const double rho[2] = {5, 6}, u[2] = {0, 0};
  for (int lattice : {MCLG_D1Q3, MCLG_D2Q9})
    for (bool b : {false, true}) {
      none = b;
      mclg_config c{};
      c.abi_version = MCLG_ABI_VERSION;
      c.lattice = (uint32_t)lattice;
      c.n_replicas = 2;
      c.L = L;
      c.Ly = Ly;
      c.lambda9 = lam;
      c.C = 2;
      c.lambda_num = c.lambda_den = 1;
      c.n_max = 40;
      REQUIRE(mclg_sizes(&c, &c.state_bytes, &c.workspace_bytes) == MCLG_OK);
      c.state = std::calloc(1, c.state_bytes);
      c.workspace = std::calloc(1, c.workspace_bytes);
      mclg_init_spec s{};
      s.kind = MCLG_INIT_POISSON;
      s.rho = rho;
      s.u0 = u;
      mclg_ctx *x = nullptr;
      REQUIRE(mclg_init(&c, &s, &x) == MCLG_OK);
      for (int k = 0; k < 2; ++k) {
        REQUIRE(mclg_step(x, 3) == MCLG_OK);
        if (lattice == MCLG_D1Q3) {
          mclg_moments_t m[2];
          REQUIRE(mclg_moments(x, nullptr, 0, 0, m) == MCLG_OK && m[0].sites == 7 && m[1].sites == 8 && m[1].t == 3 * (k + 1));
        } else {
          mclg_moments9_t m[2];
          REQUIRE(mclg_moments9(x, m) == MCLG_OK && m[0].sites == 7 && m[1].sites == 8);
        }
      }
      REQUIRE(mclg_destroy(x) == MCLG_OK);
      std::free(c.state);
      std::free(c.workspace);
    }
  std::puts("ok");
}
"""


def test_moments_without_pinned_memory(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-o", str(exe), str(src)] + [os.path.join(CSRC, f) for f in ("api.cpp", "d2q9.cpp", "regplan.cpp", "tables.cpp")],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
