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

// Tile shape, from about half of the capacity live (what a packed stream has).  Measured times: a 128 x 128 x 64 step
// takes 0.6 us alone on its unit, and the launch 3.3 us before the first and after the last; .95 and 5.5 us beside another,
// 1.65 where some units have a third tile to take and 0.0026 us per tile of the launch beyond.  A round of the large tiles
// (gemm_rows.h) takes 5 us and 1.2 a step (192) or 9.5 and 1.2 (256).  In us, called again and again, 128 | large: 6272 x 2304, K 768
// 30.1 | 25.6; 6272 x 768 14.4 | 16.3; 12544 x 768 24.5 | 22.9; 12544 x 1536, K 512 28 | 32.8; 12544 x 768, K 2304 60.5 | 52.2.  Large
// where they tie: the same launch loses in a step what it wins alone (9408 x 2304, K 768, 44.5 | 44.5, the training step around it
// 300 | 293).  A capacity of one row counts as one.
inline bool large_tiles(int m_cap, bool counted, int ncols, int kc) {      // counted: the live rows are counted on the device
  const int live = counted ? std::max(m_cap / 2, 1) : m_cap;
  const auto tiles = [&](long edge) { return gemm_tiles<long>(live, ncols, edge); };
  const auto rounds = [&](long edge) { return (double)((tiles(edge) + 255) / 256); };
  const double nk = (kc + 63) / 64, t = (double)tiles(128);                  // (contraction steps of 64)
  const double small = t <= 256 ? 3.3 + 0.6 * nk : 5.5 + nk * (t <= 512 ? 0.95 : std::max(1.65, 0.0026 * t));
  const double big = medium_tiles(live, ncols) ? rounds(192) * (5.0 + 1.2 * nk) : rounds(256) * (9.5 + 1.2 * nk);
  return big < 1.03 * small;
}

}  // namespace spa
