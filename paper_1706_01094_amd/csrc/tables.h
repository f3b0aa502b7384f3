// Host-side exact tables of the MCLG library.
//
// Collision tables: for every fiber (N, |J|) with N <= n_max and every
// incoming rest count n0, the law of n0' after C sub-collisions (or the
// fiber equilibrium for C = infinity), quantised to uint32 thresholds.
// Poisson tables: the initial-state thresholds.  See mclg.h for the rules.
#pragma once
#include <cstdint>
#include <memory>
#include <vector>

namespace mclg {

// Device image of the collision tables (copied verbatim to the workspace).
//   rowdesc[collision_row(N, n0, min(n_-1, n_+1))] = {thr offset,
//     k_first | q << 16} (device.h states the order of the rows)
//   thr[offset .. offset + q - 2] ascending uint32 thresholds
// Sampling: n0' = ((N - |J|) & 1) + 2 (k_first + #{i : thr[offset + i] <= r}).
struct CollisionTables {
  int32_t C = 0;
  uint32_t lam_p = 1, lam_q = 1, n_max = 0;
  bool galilean = false;          // per-fiber lambda of galilean_lambda_q
  std::vector<uint32_t> rowdesc;  // pairs (offset, k_first | q << 16)
  std::vector<uint32_t> thr;
  uint32_t max_q = 0;             // largest number of outcomes in a row
  // The same rows as 64 bytes of 16-bit values, each with bit 15 set: k_first,
  // then the top 15 bits of the q - 1 thresholds, padded with 0x7FFF (when
  // max_q <= 32).  A draw r whose top 15 bits equal none of them is decided by
  // the row alone: a threshold with smaller top bits is <= r, one with larger
  // top bits is > r.
  std::vector<uint16_t> row16;    // empty when not built
};

// Build (or fetch from the process cache) the tables for (C, lambda, n_max),
// with the Galilean-invariant per-fiber lambda when `galilean` is set.
// Returns nullptr for invalid parameters.
std::shared_ptr<const CollisionTables> collision_tables(int32_t C, uint32_t lam_p,
                                                        uint32_t lam_q, uint32_t n_max,
                                                        bool galilean);

// Full-fiber thresholds (uint64, 2^32 = "never") of one row, for inspection.
bool collision_row_full(int32_t C, uint32_t lam_p, uint32_t lam_q, bool galilean, uint32_t N,
                        uint32_t absJ, uint32_t n0, std::vector<uint64_t> &thr);

bool params_ok(int32_t C, uint32_t lam_p, uint32_t lam_q, uint32_t n_max, bool galilean);

// Galilean-invariant acceptance of fiber (N, |J|) for lambda~ = num / den, as
// a numerator over 2^32: floor(floor(2^32 N / sqrt(N^2 + 3 J^2)) num / den)
// (exact integer arithmetic; 2^32 num / den for J = 0).
uint64_t galilean_lambda_q(uint32_t num, uint32_t den, uint32_t N, uint32_t absJ);

// Equilibrium means of Eq. (D1Q3equil) with the stated IEEE evaluation order.
void feq(double rho, double u, double out[3]);

// Poisson(mu) thresholds of the initial-state rule (full list, uint64).
bool poisson_full(double mu, uint32_t &k_lo, std::vector<uint64_t> &thr);

// LDS image of the hottest collision rows of one workload (a performance
// cache: every site it cannot decide goes to the exact global tables, so the
// results never depend on it).
//
// A row is addressed by (a', b, c') = (min(n_-1, n_+1), n_0, max(n_-1, n_+1)),
// which fixes N, |J| and n0.  With np pairs in the image, records come in
// np + 1 rows of nb + 1: row p holds the pair's records for b = b_lo ..
// b_lo + nb - 1, then one never record; row np is all never records.  `dir`
// holds (dim_a + 1) x (dim_c + 1) entries: dir[a' (dim_c + 1) + c'] is the
// byte offset of the first record of an (a', c') pair (from the start of the
// image, whose directory comes first), that of row np for an absent pair, and
// row dim_a and column dim_c are absent pairs, so that a site's record is at
// dir[min(a', dim_a) (dim_c + 1) + min(c', dim_c)] + 16 min(b - b_lo mod
// 2^16, nb) without a range test.
//
// A record is eight uint16, of which T_j stands at {0, 2, 3, 4, 5, 6, 7, 1}[j]:
// T_j = 2^15 + the top 15 bits of thr_{k_s - 1 + j} (thr_{< 0} = 0, thr_{>=
// m - 1} = 2^32 clamped).  With rh the top 15 bits of a draw the outcome is
// state k_s + #{T_j - 2^15 < rh} - 1 when that number is at least 1 and at
// most the window's length, and no T_j - 2^15 equals rh.
//   fixed (0 < C <= 20): k_s = (b >> 1) - 3, all eight T_j: the window of the
//     moves 3 .. -3 of n0 by -2.  At rho = 50, C = 10 it misses 0.11 % of the
//     draws of its pairs, where six moves wherever they hold the most miss
//     0.30 %: near equilibrium the law is centred on no move.
//   else: k_s is the window of six moves with the most mass, T_7 holds
//     (b >> 1) - k_s as int16.  With more sub-collisions the law leaves the
//     incoming count (C = 30 at rho = 30: six moves 1.1 %, seven fixed ones
//     1.4 %; C = infinity 1.7 % and 4.8 %).
// Never records hold T_j = 2^15 only and decide nothing: the exact global row
// decides.  A pair with N < 2 (no collision) gets records of move 0.  Without
// room for any pair the image is a one-entry directory and two never records
// (np = 0, nb = 1).
struct LdsImage {
  uint32_t dim_a = 0, dim_c = 0, b_lo = 0, nb = 0;
  bool fixed = false;
  std::vector<uint32_t> dir;      // (dim_a + 1) * (dim_c + 1)
  std::vector<uint16_t> records;  // 8 per record
  double coverage = 0.0;          // expected fraction of site updates decided in LDS
  // serialised: dir padded to 16 bytes, then the records
  std::vector<uint8_t> blob() const;
  uint32_t dir_bytes() const {
    return (uint32_t)(((dim_a + 1) * (dim_c + 1) * 4 + 15) / 16 * 16);
  }
};

// Build the image for a lattice near the product-Poisson law at
// f^eq(rho, u) within `budget` bytes.
LdsImage build_image(const CollisionTables &tab, double rho, double u, uint32_t budget);

// Compacted form used on the device: n = k_first + #{thr[i] <= r}.
struct CompactLaw {
  uint32_t k_first = 0;
  std::vector<uint32_t> thr;  // q - 1 values, all < 2^32
};
CompactLaw compact(uint32_t k_lo, const std::vector<uint64_t> &full);

}  // namespace mclg
