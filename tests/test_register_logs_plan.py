"""Which calls of mclg_step_log sum their logs within launches of several steps,
and which take every interval by itself (host side, compiled here): every choice
here was timed both ways."""
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
static bool within(uint64_t L, uint64_t every, uint64_t n_logs, uint32_t n_modes = 0, bool digest = false) {
  const double coverage = 0.9971;
  const float cost = site_cost(coverage);
  const UnitPlan P = plan_units(&L, 1, 256, &cost);
  const std::vector<RegWay> ways = plan_ways(P, &L, 1, 256, true, false, true, 0.0, &cost);
  return pick_log_way(ways, every, n_logs, L, n_modes, digest, single_step(L, 1, true, 1.0 - coverage, true)) != nullptr;
}
#define REQUIRE(x) if (!(x)) { std::printf("%s\n", #x); return 1; }
int main() {
  const uint64_t M = 1 << 20;
  for (uint64_t L : {8 * M, 16 * M, 32 * M, 64 * M, 128 * M})
    for (uint64_t every : {1, 2, 3, 5}) REQUIRE(!within(L, every, 1));
  for (uint64_t L : {16 * M, 32 * M, 64 * M, 128 * M}) REQUIRE(!within(L, 1, 4));
  for (uint64_t L : {32 * M, 64 * M, 128 * M}) REQUIRE(!within(L, 1, 16) && !within(L, 10, 1));
  REQUIRE(within(128 * M, 2, 8) && within(64 * M, 2, 8) && within(128 * M, 3, 6) && within(16 * M, 1, 16));
  REQUIRE(within(4 * M, 20, 8) && within(4 * M, 20, 8, 1) && within(32 * M, 3, 6, 1) && !within(16 * M, 1, 16, 1));
  REQUIRE(within(16 * M, 10, 16) && within(8 * M, 3, 6, 1) && within(8 * M, 1, 16, 0, true));
  for (uint64_t L : {100ul, 1000ul, 4000ul, 65536ul, 1 * M, 4 * M})
    REQUIRE(within(L, 1, 16) && within(L, 1, 16, 1) && within(L, 10, 16, 1) && within(L, 10, 25));
  std::puts("ok");
}
"""


def test_logs(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-o", str(exe), str(src), os.path.join(CSRC, "regplan.cpp")], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
