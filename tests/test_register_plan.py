"""How lattices are laid out for the kernels that hold sites in registers
(host side, compiled here): every lattice is covered once, parts meet the
kernels' limits, and the parts' strips join neighbours."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(__file__)), "paper_1706_01094_amd", "csrc")

MAIN = r"""
#include <cstdio>
#include <random>
#include "regplan.h"
using namespace mclg;
// (in the kernels' file, which needs a device compiler)
namespace mclg {
bool reg_has(uint32_t Q, bool galilean, bool fixed, bool logs) {
  if (logs) return !galilean && fixed && Q <= 4;
  return fixed ? !galilean || Q <= 2 : Q == 2;
}
}
#define REQUIRE(x) if (!(x)) { std::printf("case %d: %s\n", c, #x); return 1; }
int main() {
  std::mt19937_64 g(7);
  for (int c = 0; c < 400; ++c) {
    const uint32_t n = c < 100 ? 1 : 1 + g() % (c % 3 ? 40 : 1500), blocks = c % 5 ? 256 : 1 + g() % 300;
    std::vector<uint64_t> L(n);
    for (auto &l : L) l = 1 + g() % (1ull << (1 + g() % (n == 1 ? 29 : 21)));
    std::vector<float> cost(n, 1.0f);
    if (c % 2) for (auto &x : cost) x = site_cost(1.0 - 0.2 * (g() % 1000) / 1000);
    for (float x : cost) REQUIRE(x >= 1.0f && x < 2.0f);
    const UnitPlan P = plan_units(L.data(), n, blocks, c % 2 ? cost.data() : nullptr);
    const uint32_t nb = blocks < kPlanBlocks ? blocks : kPlanBlocks;
    REQUIRE(P.first.size() == nb + 1 && P.first[0] == 0 && P.first[nb] == P.units.size());
    REQUIRE(P.units.size() <= max_units(n) && P.strips.size() <= kMaxStrips);
    std::vector<uint64_t> seen(n, 0);
    for (const UnitDev &u : P.units) {
      REQUIRE(u.slot < n && u.x0 < u.x1 && u.x1 <= L[u.slot]);
      REQUIRE(u.x0 % 8 == 0 && (u.x1 % 8 == 0 || u.x1 == L[u.slot]));
      seen[u.slot] += u.x1 - u.x0;
      if (!u.split) { REQUIRE(u.x0 == 0 && u.x1 == L[u.slot]); continue; }
      REQUIRE(u.x1 - u.x0 >= kMaxHalo && u.el < P.strips.size() && u.er < P.strips.size());
      REQUIRE(P.strips[u.er].slot == u.slot && P.strips[u.er].x == u.x1);
      REQUIRE(P.strips[u.el].slot == u.slot && P.strips[u.el].x == (u.x0 ? u.x0 : L[u.slot]));
    }
    // (lattices too short for tiles are no units)
    for (uint32_t r = 0; r < n; ++r) REQUIRE(seen[r] == (L[r] < kMinTiled ? 0 : L[r]));
    for (const RegWay &w : plan_ways(P, L.data(), n, blocks, c % 2, c % 7 == 0, c % 11 != 0, c % 3 ? 0.05 : 0.3,
                                        c % 2 ? cost.data() : nullptr)) {
      REQUIRE(w.kind != RegWay::kNone && w.most >= 1 && w.step_us > 0 && w.launch_us > 0);
      REQUIRE(reg_has(w.Q, c % 7 == 0, c % 11 != 0, w.logs));
      REQUIRE(w.Q != 6 || c % 3);
      uint64_t longest = 0;
      bool ragged = false;
      for (uint64_t l : L) { longest = l > longest ? l : longest; ragged |= l % 8 != 0; }
      if (w.kind == RegWay::kRing) {
        REQUIRE(longest <= 4096ull * w.Q && (w.team == 0 || (longest <= 256ull * w.Q && w.team <= 16)));
      } else {
        // a tile's positions fit a wave and, with its extra sites, the lattice
        REQUIRE(2 * w.kh < 256 * w.Q && w.kh <= kMaxHalo && w.kh % 8 == 0);
        REQUIRE(w.most + (ragged ? 8 : 0) <= w.kh && P.n_long > 0 && P.units.size() >= P.n_long);
        REQUIRE(!w.logs || n == 1);
      }
    }
  }
  std::puts("ok");
}
"""


def test_units_and_ways(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    "-o", str(exe), str(src), os.path.join(CSRC, "regplan.cpp")], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
