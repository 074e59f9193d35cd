// The tile shapes of the row GEMM (gemm_rows.h) and the rules that choose among them; no device code, so that a host
// program can ask them.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

namespace spa {

template <class T>
__host__ __device__ inline T gemm_tiles(T rows, T ncols, T edge) { return (rows + edge - 1) / edge * ((ncols + edge - 1) / edge); }
__host__ __device__ inline bool medium_tiles(int rows, int ncols) {
  return 7 * ((gemm_tiles(rows, ncols, 192) + 255) / 256) <= 10 * ((gemm_tiles(rows, ncols, 256) + 255) / 256);
}
// The large shapes of a launch: 192 x 192 for all rows, or 256 x 256 for the first wide_rows and 256 x 192 for the others.  Chosen by
// the units' rounds: one of 192 x 192 takes .7 and one of 256 x 192 .83 of one of 256 x 256 (K 768: 15.5 to 18.5 | 19.5 to 20.6 | 21.6 to
// 25 us; K 2304: 47 | 53 | 61).  Where more than a round is due the last rows go to 256 x 192 if that saves a part of one (12544 rows
// of 2304 columns: 1.83 instead of 2 rounds, 47.4 instead of 51 us).  Units without a tile in a single round clear or copy the rows of
// out that no packed row maps to beside the others, ten rows of 768 columns a us each; what they cannot do comes after the tiles (13500 rows of 768
// columns with the residual: 256 x 192 would leave 44 units for the copy, 36 us, 256 x 256 leaves 97, 34.5).
struct LargePlan {
  bool medium;
  int wide_rows, rounds, rest;   // rounds of the units: of 192 x 192 or 256 x 256, and of 256 x 192
};
// What the choice takes from the call, formed on the host (a division by a value of the call costs the device a tenth of a
// microsecond): rows of 256 x 256 tiles in a round; rows of out that a wave without a tile clears, or copies, while the others
// multiply; what any and what each row left to the units with a tile costs, in hundredths of a round (1 us, and 5 TB/s).
struct LargeRule {
  int wide, fit, late;
  float left;
};
inline LargeRule large_rule(int ncols, int kc, bool copy) {
  const int nk = std::min((kc - 1) / 64 + 1, 10000), bytes = std::min(ncols, 1 << 24) * (copy ? 4 : 2), row = std::min(ncols, 1 << 24) * 4;
  return {256 / ((ncols + 255) / 256), std::clamp((4 + nk) * 5120 / row, 1, 100000), 100 / (8 + nk), bytes / (50000.f * (8 + nk))};
}
// more: rows of out to clear or copy beside the products.
__host__ __device__ inline LargePlan large_plan(int rows, int ncols, int more, const LargeRule& rule) {
  const auto rounds = [](int tiles) { return (tiles + 255) / 256; };
  const int t192 = gemm_tiles(rows, ncols, 192);
  // The cheapest there is.  (Every workgroup forms the plan before its first load, half a microsecond for the rest of it: 9555 live rows of 192 -> 576
  // 9.1 us without this exit, 8.75 with it, 8.6 with a rule of two shapes.)
  if (t192 <= 256 && more <= 0) return {true, 0, rounds(t192), 0};
  const int mt = (rows + 255) / 256, n256 = (ncols + 255) / 256, n192 = (ncols + 191) / 192;
  // what the units left over in a single round do not clear or copy
  const auto after = [&](int tiles) {
    const int left = more - (tiles < 256 ? (256 - tiles) * 8 * rule.fit : 0);
    return left > 0 ? rule.late + (int)((float)left * rule.left) : 0;
  };
  LargePlan plan = {true, 0, rounds(t192), 0};
  int cost = 70 * plan.rounds + after(t192);
  if (!medium_tiles(rows, ncols)) plan = {false, rows, rounds(mt * n256), 0}, cost = 100 * plan.rounds + after(mt * n256);
  const int full = mt * n256 / 256;                    // full rounds of 256 x 256
  for (int i = 0; i < 3; ++i) {
    const int r = i == 0 ? 0 : full + 1 - i, wide = r * rule.wide, tiles = (mt - wide) * n192;
    if (r < 0) continue;
    const int c = 100 * r + 83 * rounds(tiles) + after(r == 0 ? tiles : 256);
    if (c < cost) {
      cost = c;
      plan = {false, wide * 256 < rows ? wide * 256 : rows, r, rounds(tiles)};
    }
  }
  return plan;
}

// Tile shape, from about half of the capacity live (what a packed stream has).  Measured times: a 128 x 128 x 64 step
// takes 0.6 us alone on its unit, and the launch 3.3 us before the first and after the last; .95 and 5.5 us beside another,
// 1.65 where some units have a third tile to take and 0.0026 us per tile of the launch beyond.  A round of the large tiles
// (gemm_rows.h) takes 5 us and 1.2 a step (192 x 192), 5 and 1.4 (256 x 192) or 9.5 and 1.2 (256 x 256).  In us, called again and again, 128 | large: 6272 x 2304, K 768
// 30.1 | 25.6; 6272 x 768 14.4 | 16.3; 12544 x 768 24.5 | 20.6; 12544 x 1536, K 512 28 | 32.8; 12544 x 768, K 2304 60.5 | 52.8.  Large
// where they tie: the same launch loses in a step what it wins alone (9408 x 2304, K 768, 44.5 | 44.5, the training step around it
// 300 | 293).  A capacity of one row counts as one.
inline bool large_tiles(int m_cap, bool counted, int ncols, int kc) {      // counted: the live rows are counted on the device
  const int live = counted ? std::max(m_cap / 2, 1) : m_cap;
  const auto tiles = [&](long edge) { return gemm_tiles<long>(live, ncols, edge); };
  const double nk = (kc + 63) / 64, t = (double)tiles(128);                  // (contraction steps of 64)
  if (t > 1 << 24) return true;
  const double small = t <= 256 ? 3.3 + 0.6 * nk : 5.5 + nk * (t <= 512 ? 0.95 : std::max(1.65, 0.0026 * t));
  const LargePlan plan = large_plan(live, ncols, 0, large_rule(ncols, kc, false));
  const double big = plan.medium ? plan.rounds * (5.0 + 1.2 * nk) : plan.rounds * (9.5 + 1.2 * nk) + plan.rest * (5.0 + 1.4 * nk);
  return big < 1.03 * small;
}

// 128 x 128 tiles one a unit (gemm_rows_ring_kernel) or two a unit.  One where three quarters of the capacity are no more tiles than
// units: a second round of single tiles costs more than neighbours that cover each other's waits.  us, one | two a unit: 1152 -> 384, 294
// tiles of capacity, 6272 rows (147 tiles) 10.9 | 13.9, 11289 rows (267) 21.5 | 19.2; 2304 -> 768 of the same capacity, 3136 rows 17.4 | 25.0;
// 441 tiles of 384 -> 1152 12.0 | 10.9, 294 of 768 -> 768 16.2 | 14.8.
inline bool ring_tiles(int m_cap, bool counted, int ncols) {
  return gemm_tiles<long>(counted ? m_cap - m_cap / 4 : m_cap, ncols, 128) <= 256;
}
// Eight waves and two steps, two a unit: where one a unit might need a second round and has few steps to gain on.  us, 19110 rows of 192 -> 192
// (300 tiles of capacity), half | nine tenths live, two a unit in four waves 5.4 | 6.9, one a unit 5.1 | 9.2, so 5.0 | 7.1; with copied rows 7.7 | 9.3, 8.1 |
// 12.7, 7.0 | 9.4; 19600 of 256 -> 256 copied 8.2 | 11.3, 8.7 | 14.1, 7.8 | 10.9; 14000 of 320 8.3 | 11.5, 9.3 | 14.2, 8.1 | 11.3.  With more steps one a
// unit gains more than a rare second round costs: 12544 of 384 9.0 | 12.5, 8.4 | 15.6, 8.9 | 12.1; 5000 of 1024 14.7 | 20.6, 11.7 | 22.4, 15.4 | 20.1.
inline bool two_rings(int m_cap, bool counted, int ncols, int kc) {
  return kc <= 320 && ring_tiles(m_cap, counted, ncols) && gemm_tiles<long>(m_cap, ncols, 128) > 256;
}

}  // namespace spa
