"""The parts that lattices between two blocks are cut into (host side, compiled
here): none shorter than the sites on each side of a tile, whatever a site of
the lattice costs and whatever lies beside it."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(__file__)), "paper_1706_01094_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include "regplan.h"
using namespace mclg;
// (in the kernels' file, which needs a device compiler)
namespace mclg {
bool reg_has(uint32_t, bool, bool, bool) { return false; }
}
static int check(const std::vector<uint64_t> &L, const std::vector<float> &cost, uint32_t blocks) {
  const UnitPlan P = plan_units(L.data(), (uint32_t)L.size(), blocks, cost.data());
  std::vector<uint64_t> seen(L.size(), 0);
  for (const UnitDev &u : P.units) {
    seen[u.slot] += u.x1 - u.x0;
    if (u.split && u.x1 - u.x0 < kMaxHalo) {
      std::printf("a part of %u sites of a lattice of %llu beside %zu, cost %g, %u blocks\n", u.x1 - u.x0,
                  (unsigned long long)L[u.slot], L.size() - 1, cost[u.slot], blocks);
      return 1;
    }
  }
  for (size_t r = 0; r < L.size(); ++r)
    if (seen[r] != L[r]) { std::printf("%llu sites of %llu\n", (unsigned long long)seen[r], (unsigned long long)L[r]); return 1; }
  return 0;
}
int main() {
  const double coverage[] = {1.0, 0.997, 0.95, 0.88, 0.5, 0.0};
  for (double cov : coverage)
    for (uint64_t L = kMinTiled; L <= 4000; ++L)
      for (uint32_t blocks : {2u, 7u, 256u})
        if (check({L}, {site_cost(cov)}, blocks) || check({20000, L}, {site_cost(1.0), site_cost(cov)}, blocks)) return 1;
  for (uint64_t L = 65000; L <= 66000; ++L)
    if (check({L}, {site_cost(0.0)}, 256)) return 1;
  std::puts("ok");
}
"""


def test_no_part_is_shorter_than_a_tiles_extra_sites(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-o", str(exe), str(src), os.path.join(CSRC, "regplan.cpp")], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
