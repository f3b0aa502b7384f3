// D2Q9 contexts of the MCLG library (host side): layout, collision rules,
// launches.  The rules and the layout are described in mclg.h.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "../../include/mclg.h"
#include "device.h"
#include "moments.h"

namespace mclg {

struct D2Ctx {
  uint32_t n = 0, flags = 0, D = 0, Dq = 0;
  uint32_t first_table = 1;  // that the step kernels read to begin with (see Step9)
  int32_t C = 0;
  uint64_t seed = 0;
  int64_t t = 0;
  std::vector<uint64_t> Lx, Ly, rid, dense;
  std::vector<Rep9> reps;
  std::vector<Tile9> tiles;
  std::vector<uint32_t> rules;      // 81 x kRule9Words
  std::vector<uint32_t> rules_dev;  // kRule9DevWords
  uint64_t state_bytes = 0, ws_bytes = 0;
  uint64_t o_err = 0, o_reps = 0, o_tiles = 0, o_rules = 0, o_pdesc = 0, o_pool = 0,
           o_dense = 0;
  MomPlan mplan;  // moment kernels: segments and runs (one per replica)
  uint64_t o_mseg = 0, o_mrun = 0, o_mslot = 0, o_mpart = 0, o_mout = 0;
  uint16_t *state = nullptr;
  uint8_t *ws = nullptr;
  hipStream_t stream = nullptr;
  long long *pin = nullptr;  // results of the moments and the error word (up to kMomPinned replicas)
  int last_hip = 0;
  ~D2Ctx() {
    if (pin) (void)hipHostFree(pin);
  }
};

// Collision rule table of mclg.h for lambda9 (18 values); false when a
// lambda is not in [0, 1], D would reach 2^32, or a source's targets would
// add up to more than one.
bool build_rules9(const uint32_t *lambda9, std::vector<uint32_t> &rules, uint32_t &D);

// The rules as the step kernel reads them: three tables, of which a block
// holds the one that its sites need.  K_j = n_0 + ... + n_j (j = 0..7).
// - wide (any N, any D), per ordered source pair p = 9 i + j, 24 words: words
//   0-3 the cumulative weights c_q; then, for q = 0..4, four words holding the
//   change of the K_j as 16-bit two's-complement pairs, K_2m in the low and
//   K_2m+1 in the high half;
// - half (N < 2^15, Dq <= 2^15, Dq = D / g with g the greatest common divisor
//   of D and all weights: a target draw u is used as floor(u / g)), per pair p, 22 words: words 0-1 the
//   halves 2^15 - c_q / g; then, for q = 0..4, four words, the 32-bit sum of the
//   changes of the halves 2^15 - K_j, times 2^16 in the high half;
// - byte (N < 2^7, Dq <= 2^15), per pair p, 14 words: words 0-1 as
//   above; then, for q = 0..4, two words of the changes of the bytes
//   2^7 - K_j alike.
constexpr uint32_t kRule9Wide = 24, kRule9Half = 22, kRule9Byte = 14;
// (each table starts at, and is read in, 16-byte pieces)
constexpr uint32_t rule9_words(uint32_t per_pair) { return (81u * per_pair + 3u) / 4u * 4u; }
constexpr uint32_t kRule9WideAt = 0, kRule9HalfAt = kRule9WideAt + rule9_words(kRule9Wide),
                   kRule9ByteAt = kRule9HalfAt + rule9_words(kRule9Half),
                   kRule9DevWords = kRule9ByteAt + rule9_words(kRule9Byte);
constexpr uint32_t kRule9MaxPacked = 1u << 15;  // Dq of the packed tables, at most
std::vector<uint32_t> device_rules9(const std::vector<uint32_t> &rules, uint32_t D, uint32_t &Dq);

// Validate a D2Q9 configuration and fill the layout (sizes and offsets).
int d2q9_layout(const mclg_config *cfg, D2Ctx &d);
int d2q9_init(D2Ctx &d, const mclg_config *cfg, const mclg_init_spec *init);
int d2q9_step(D2Ctx &d, uint64_t n_steps);
int d2q9_get_counts(D2Ctx &d, uint32_t r, uint16_t *out);
int d2q9_moments(D2Ctx &d, mclg_moments9_t *out);
int d2q9_check(D2Ctx &d);
int d2q9_histogram(D2Ctx &d, uint32_t n_bins, uint64_t *dev_hist);

}  // namespace mclg
