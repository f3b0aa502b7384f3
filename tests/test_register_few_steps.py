"""Which calls of few steps take one step per launch (host side, compiled here):
a launch of tiles is never taken for one step, nor, on large or crowded
lattices and with the dearer rules, for two or three; longer calls and smaller
lattices keep theirs.  Every choice here was timed both ways."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(__file__)), "paper_1706_01094_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "regplan.h"
using namespace mclg;
// (in the kernels' file, which needs a device compiler)
namespace mclg {
bool reg_has(uint32_t Q, bool galilean, bool fixed, bool logs) {
  if (logs) return !galilean && fixed && Q <= 4;
  return fixed ? !galilean || Q <= 2 : Q == 2;
}
}
static bool reg(std::vector<uint64_t> L, uint64_t steps, double coverage, bool galilean = false, bool fixed = true,
                bool one_image = true) {
  const std::vector<float> cost(L.size(), site_cost(coverage));
  uint64_t sites = 0;
  for (uint64_t l : L) sites += l;
  const uint32_t n = (uint32_t)L.size();
  const UnitPlan P = plan_units(L.data(), n, 256, cost.data());
  const std::vector<RegWay> ways = plan_ways(P, L.data(), n, 256, one_image, galilean, fixed,
                                             crowded_image(coverage) ? 1.0 : 0.0, cost.data());
  return pick_way(ways, steps, single_step(sites, n, one_image, 1.0 - coverage, fixed)) != nullptr;
}
#define REQUIRE(x) if (!(x)) { std::printf("%s\n", #x); return 1; }
int main() {
  const double rho15 = 0.9998, rho50 = 0.9971, rho100 = 0.897, c30 = 0.9705;
  const uint64_t M = 1 << 20;
  for (double cov : {rho15, rho50, rho100, 0.0})
    for (uint64_t L : {16 * M, 24 * M, 32 * M, 48 * M, 64 * M, 100 * M, 128 * M, 64 * M + 3})
      REQUIRE(!reg({L}, 1, cov));
  REQUIRE(!reg(std::vector<uint64_t>(1024, 131000), 1, rho50) && reg(std::vector<uint64_t>(1024, 131000), 2, rho50));
  REQUIRE(!reg({24 * M}, 2, rho50) && !reg({32 * M}, 2, rho50) && reg({32 * M}, 2, rho15) && reg({32 * M}, 2, rho100));
  REQUIRE(reg({64 * M}, 2, rho15) && reg({64 * M}, 2, rho50) && !reg({64 * M}, 2, rho100) && reg({64 * M}, 3, rho100));
  REQUIRE(!reg({16 * M}, 3, rho50, true) && !reg({16 * M}, 4, rho50, true) && reg({16 * M}, 6, rho50, true));
  REQUIRE(!reg({64 * M}, 2, rho50, true) && !reg({64 * M}, 3, rho50, true) && reg({64 * M}, 4, rho50, true));
  REQUIRE(!reg({16 * M}, 6, c30, false, false) && reg({16 * M}, 12, c30, false, false));
  REQUIRE(!reg(std::vector<uint64_t>(300, 20000), 2, 0.9993) && reg(std::vector<uint64_t>(300, 20000), 3, 0.9993));
  REQUIRE(reg(std::vector<uint64_t>(2000, 30000), 2, 0.98, false, true, false));
  // small lattices from the first step on, and all from a few
  REQUIRE(reg({1000}, 1, rho50) && reg({100}, 1, rho50) && reg(std::vector<uint64_t>(19, 100), 1, rho50));
  for (double cov : {rho15, rho50, rho100})
    for (uint64_t L : {64ul, 1000ul, 65536ul, 1000003ul, 4 * M, 16 * M, 64 * M, 128 * M})
      for (uint64_t k : {3, 8, 64, 1000}) REQUIRE(reg({L}, k, cov));
  std::puts("ok");
}
"""


def test_few_steps(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-o", str(exe), str(src), os.path.join(CSRC, "regplan.cpp")], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
