// Rules that choose a product's kernel and its shape, in plain C++ (no HIP), so
// that they can be checked on the host.
#pragma once

#include <stdint.h>

namespace oq {

// Shape of the small-M (weight-streaming) product: 16 nb columns a workgroup
// of `waves` waves, and ub 128-code units of K that a wave loads a round.
// 32 columns when N is wide enough to keep more than 256 workgroups busy, else
// 16; waves sized so that each takes one or two units at K <= 1024, and two
// (16 columns) or four (32 columns) in a round above; deeper K runs more
// rounds.  A round loads ub units whether the wave has them or not, so up to K
// = 2048, two units for each of 8 waves and one for each of 16, the rounds are
// that short (5 x 32768 x 2048: 11.4 -> 7.1 us), and K = 64, whose rows hold
// half a unit, loads none and leaves its 64 codes to the last 64-code step.
// 8-bit token codes take twice the registers per unit: half the units a round
// in the deep cases (1024 threads leave 128 registers per lane).
struct SmallShape {
  int nb, waves, ub;
};
constexpr SmallShape small_shape(int64_t N, int64_t K, bool a8) {
  if (N > 4096) return {2, 8, K < 128 ? 0 : K <= 1024 ? 1 : K <= 2048 || a8 ? 2 : 4};
  return {1, K <= 1024 ? 4 : 16, K < 128 ? 0 : K <= 1024 ? 2 : K <= 2048 || a8 ? 1 : 2};
}

}  // namespace oq
