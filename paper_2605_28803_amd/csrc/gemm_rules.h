// Rules that choose a product's kernel and its shape, in plain C++ (no HIP), so
// that they can be checked on the host.
#pragma once

#include <stdint.h>

namespace oq {

// Whether the small-M (weight-streaming) kernel takes a product; the LDS-tiled
// ring takes the others.  a8: 8-bit token codes; tiled: token codes in the
// 16-row tiled layout, which only the small-M kernel reads (row groups of 64
// along grid.y when M > 64).
//
// Row-layout codes: up to M = 16, and up to M = 64 while N <= 8192.  A
// workgroup re-reads every token code for its 32 columns in operand order (16
// rows of 64 bytes a load), which above one row block costs more than the
// weight stream once the columns are many.  Weights from HBM, us on the small-M
// kernel against the ring: 40 x 32768 x 2048 29.2 / 11.6, 17 x 9000 x 4096 13.9 /
// 11.1, 64 x 10000 x 8192 31.7 / 19.5; 17 x 8192 x 8192 11.8 / 13.2; one row block, 1 and
// 16 x 16384 x 16384: 29.9 / 37.9 and 34.8 / 39.0 (with weights that stay in the cache
// the ring is 2 us ahead there).
// Between 8192 and 16384 columns the ring has at most one 64 x 64 tile per CU,
// so its time is a tile's whole K, and with few rows the small-M kernel stays
// ahead where its own K loop is short or the ring's long:
//  * K = 64, one step on either: 17 x 8200 x 64 2.8 / 3.1, 48 x 9000 x 64 3.4 / 3.4, 64 x
//    9000 x 64 3.7 / 3.4; W4A8, whose ring has no short stages, 64 x 9000 x 64 3.8 / 4.2.
//  * up to K = 1024, where a wave loads all it needs at once (above, it takes a
//    second round).  The ring's stages are 512 codes (up to K = 256: 128; 8-bit
//    tokens: 256), so it is ahead at a whole number of them: W4A4 17 x 8200 x 128 3.4 / 3.3,
//    x 192 3.5 / 3.6, x 384 3.6 / 4.1, x 512 4.0 / 4.3 but 32 x 8200 x 512 4.5 / 4.3, 40 x 12288 x 448 4.3 / 4.4,
//    64 x 8200 x 640 4.3 / 5.2, 64 x 16384 x 896 5.9 / 6.2, 64 x 9000 x 832 6.0 / 5.8, 40 x 12288 x 1024 5.7 / 5.7, 48 x
//    9000 x 1024 5.7 / 5.5; W4A8 24 x 8200 x 320 4.6 / 4.3, 40 x 8200 x 576 4.9 / 5.0, 24 x 12288 x
//    576 5.2 / 5.5, x 768 5.9 / 5.5, 24 x 8200 x 640 4.9 / 4.7, 48 x 16384 x 832 6.7 / 6.8, 24 x
//    9000 x 896 5.3 / 5.2, 17 x 8200 x 1024 5.1 / 5.9, 28 x 9000 x 1024 6.2 / 6.0.
//    A second tile for some CUs leaves that so up to 24576 columns, for fewer rows:
//    W4A4 48 x 20000 x 640 6.7 / 7.1, 17 x 20000 x 704 6.5 / 6.8, 17 x 16392 x 1024 5.9 / 6.3, but
//    17 x 32768 x 640 7.3 / 7.1.
//  * deep K of W4A8, whose tile takes twice the LDS reads: 17 x 8200 x 8192 25.9 /
//    28.6, 17 x 8200 x 16384 43.4 / 53.3, 28 x 8200 x 16384 49.9 / 53.6, 17 x 16384 x 16384 53.5 /
//    58.1; but 24 x 9000 x 8192 30.6 / 28.9, 24 x 10000 x 16384 54.8 / 53.6.
constexpr bool few_rows(int64_t M, int64_t N, int64_t K, bool a8, bool tiled) {
  if (tiled || M <= 16) return true;
  if (M > 64) return false;
  if (N <= 8192) return true;
  if (N > 16384) {
    if (a8 || N > 24576 || K <= 512 || K > 1024) return false;
    return M <= (K % 256 == 128 ? 48 : K % 256 ? 32 : 20);
  }
  if (K == 64) return a8 || M <= 48;
  if (a8) {
    if (K == 576 || K == 704) return M <= (N < 9000 ? 40 : 24);
    if (K == 640 || K == 768) return N < 9000 && M <= 20;
    if (K == 832 || K == 960) return N < 9000 || M <= 48;
    if (K == 896 || K == 1024) return M <= (N < 9000 ? 40 : 24);
    return (K >= 4096 && N < 9000 && M <= (K > 8192 ? 28 : 24)) || (K > 8192 && M <= 20);
  }
  if (K == 192) return N < 9000 && M <= 32;
  if (K <= 256 || K > 1024) return false;
  if (K < 512) return N < 9000 || M <= 40;
  if (K == 512) return N < 9000 && M <= 24;
  if (K % 256 == 0) return M <= (N < 9000 ? 48 : 40);
  return K < 768 || K == 896 || N < 9000 || M <= 56;
}

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

// The ring's tilings.  Estimated time of one: fixed + (rounds - 1) * 2 us + K *
// (one tile on a CU: lat; n tiles sharing a CU: n * thr), lat and thr in ns per code
// of K; occ: workgroups per CU.  Against the times of every tiling at sixteen shapes
// from 128 x 4096 x 4096 to 16384 x 8192 x 8192, which the host test of this rule holds,
// the estimates are 0.79 to 1.03 of the measured time for W4A4, but up to 1.39 for
// 256 x 256 tiles that do not fill the chip (nothing else would take them there), and
// 0.86 to 1.28 for W4A8.  The tiling chosen is the fastest or within 7% of it at all of
// them but one (W4A8 816 x 2560 x 2048: 18%).
struct RingCost {
  int bm, bn, occ;
  float lat, thr, fixed;
};
constexpr RingCost kRingCost[] = {{256, 256, 1, 12.5f, 11.9f, 8.0f},  // 8 waves of 128 x 64, 256-code stages
                                  {128, 128, 2, 3.4f, 3.35f, 4.6f},   // 4 waves of 64 x 64
                                  {128, 64, 3, 2.45f, 1.92f, 3.9f},   // 4 waves of 64 x 32
                                  {64, 64, 2, 0.9f, 1.0f, 5.4f},      // 4 K groups of 2 waves of 64 x 32, 512-code stages
                                  {64, 64, 2, 1.45f, 1.15f, 3.7f}};   // 4 waves of 32 x 32, 512-code stages
constexpr RingCost kRingCostA8[] = {{256, 256, 1, 14.2f, 14.3f, 8.0f},   // 8 waves of 128 x 64, 128-code stages
                                    {128, 128, 2, 5.1f, 4.35f, 4.5f},    // 4 waves of 64 x 64
                                    {64, 64, 2, 2.2f, 1.6f, 4.4f}};      // 2 K groups of 2 waves of 64 x 32
constexpr float ring_estimate(const RingCost& c, int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
  const int64_t n = (tiles + 255) / 256, rounds = (n + c.occ - 1) / c.occ;
  const float k = 1e-3f * static_cast<float>(K);
  return c.fixed + 2.0f * static_cast<float>(rounds - 1) + k * (n == 1 ? c.lat : static_cast<float>(n) * c.thr);
}
// Index of the tiling.  K <= 256, W4A4: 5 or 6, 64 x 64 and 128 x 64 tiles of 4
// waves with 128-code stages.  There a tile is one or two stages; the others'
// 256- and 512-code stages load and multiply what is not there, and their two
// buffers leave room for fewer workgroups a CU, while such a product is bound by
// its output stores, which want many in flight.  64 x 64 as long as a CU gets three
// of them, us against the best of the others: 65 x 16384 x 128 5.5 -> 4.2,
// 600 x 4096 x 128 5.8 -> 4.8;
// above, 128 x 64: 4080 x 4096 x 64 14.0 -> 11.7, 8192 x 8192 x 256 44.4 -> 37.0.
// W4A8 up to K = 256: no 256 x 256 tiles while a CU gets at most five of them, for
// the same reason: 1100 x 32768 x 128 32.1 us, with 128 x 128 25.8; 2500 x 32768 x 256 60.6 / 56.3; but
// 4080 x 32768 x 128 90.5 / 102.
// Else the one with the lowest estimate.
constexpr int ring_tiling(int64_t M, int64_t N, int64_t K, bool a8) {
  if (!a8 && K <= 256) return ((M + 63) / 64) * ((N + 63) / 64) <= 768 ? 5 : 6;
  const RingCost* c = a8 ? kRingCostA8 : kRingCost;
  const int count = a8 ? 3 : 5;
  int best = a8 && K <= 256 && ((M + 255) / 256) * ((N + 255) / 256) <= 1280 ? 1 : 0;
  for (int i = best + 1; i < count; ++i)
    if (ring_estimate(c[i], M, N, K) < ring_estimate(c[best], M, N, K)) best = i;
  return best;
}

}  // namespace oq
