// How the weight side of the projections' backward (linear_bwd.hip) is cut: tile edge and chunks of tokens; no device code, so
// that a host program can ask the rules.
#pragma once

#include <algorithm>
#include <cmath>

#include "gemm_shape.h"

namespace spa {

constexpr int kWeightEdge = 128;

// Tiles of `edge`, `splits` chunks of tokens.  The number of chunks and `fold` decide the bits of the result, the edge does not.
struct WeightShape {
  int edge, splits;
  bool fold = false;             // a chunk's sums of every 256 rows are added up apart (128 x 128 tiles)
  long tiles(int n_out, int K) const { return gemm_tiles<long>(n_out, K, edge); }
};

// Number of token chunks.  It decides the bits of the result, so it follows from the call alone, whatever stands beside it in
// a group; `forced` (option gemm_splits) overrides it.
// With 128 x 128 tiles: (chunk, tile) workgroups for two per compute unit (what is resident at a time), at most 16
// chunks (every chunk's partial tiles are written and read once), chunks of at least 256 rows at full capacity, and
// one chunk (no partial tiles, no second launch) up to 2048 rows: at half of them live its 16 steps take as long as 3
// steps and the second launch.
inline int weight_splits(int M_cap, int K, int N_out, int forced) {
  if (forced > 0) return forced;
  const long tiles = gemm_tiles<long>(N_out, K, kWeightEdge);
  if (M_cap <= 2048) return 1;
  const long by_rows = std::max(M_cap / 256, 1);
  return (int)std::clamp(std::min(512 / tiles, by_rows), 1L, 16L);
}
// With 256 x 256 tiles: a workgroup a unit, chunks of at least 512 rows at full capacity.
inline int weight_splits_big(int M_cap, long tiles, long most, int forced) {
  if (forced > 0) return forced;
  const long by_rows = std::max(M_cap / 512, 1);
  return (int)std::clamp(std::min(256 / tiles, by_rows), 1L, most);
}
// The weight sides of a block (N_out = K and 3 K) stand in one group.  Up to a line they share a launch of 128 x 128 tiles with the input
// side; beyond, the two alone have one of 256 x 256 tiles on a second stream (or in order), which they fill together with fewer chunks than
// each by itself (12544 live rows, 768 columns: seven; with their sums 84.7 us, as two launches of 128 x 128 tiles and one for the sums 93).  More
// than ten do not pay (a step of 25088 rows, 512 columns, 10 | 16: 237.8 | 238.8 us; 32768 rows 279.6 | 284.8).
constexpr double kPairWork = 2.4e10;                       // multiplications of both
inline double weight_work(int M_cap, int K, int N_out) { return (double)M_cap * K * N_out; }
// The line.  One launch saves the streams' events and a launch, a constant; a second stream has the gate backward, whose time goes with rows x
// columns, beside the weight sides, so that narrow blocks of many rows pass to it earlier.  us a training step, one launch | second stream: 12152
// rows of 768 columns (7.2e9) 192.7 | 202.4, 9016 of 896 (7.2e9) 187.8 | 196.3, 17836 of 640 (7.3e9) 215.6 | 214.3, 16464 199.1 | 202.6, 21560 of 576 (7.2e9)
// 232.6 | 228.3, 23912 of 512 (6.3e9) 197.7 | 199.6; 25600 of 512 (6.7e9) 205.6 | 205.6, 27648 (7.2e9) 230.0 | 214.3, 27648 of 480 (6.4e9) 234.7 |
// 223.6, 32768 of 448 (6.6e9) 227.5 | 220.0, 48640 of 384 (7.2e9) 277.4 | 277.6; 29400 of 448 (5.9e9) 219.2 | 221.7.  (Blocks of 768 columns and more would
// gain up to 9.2e9: 13328 rows of 768 205.1 | 209.4, 15680 231.6 | 231.5, 8624 of 1024 216.5 | 226.9.)
inline bool in_one_launch(int M_cap, int C) { return weight_work(M_cap, C, C) <= (M_cap <= 24000 ? 7.3e9 : 6e9); }
inline bool of_a_block(int K, int N_out) { return N_out == K || N_out == 3 * (long)K; }
// The chunks that a call would have for speed alone.  Where a block's have fewer, and in no tile that cannot add up sums apart (256 x 256
// has no registers for a second sum), the sums are added up apart.
inline int weight_most_splits(int M_cap, int K, int N_out, int forced) {
  if (of_a_block(K, N_out) && 4 * weight_work(M_cap, K, K) > kPairWork)
    return weight_splits_big(M_cap, gemm_tiles<long>(K, K, 256) + gemm_tiles<long>(3L * K, K, 256), 10, forced);
  return weight_splits(M_cap, K, N_out, forced);
}
// The chunks of a block's sides in the one launch: a chunk more shortens the walk over the rows and writes and reads a partial result more, which
// come out even where the number is as sqrt(rows) / columns; the factor is that of the best steps measured, with 1 to 16 chunks.  us a training step of
// a block, with as many as fill the chip | so: 3136 rows of 1024 columns of capacity 136 | 122 (1 chunk), 5096 165 | 150 (1), 3136 of 768
// 111 | 103 (1), 6272 140 | 132 (2), 9408 167 | 164 (2), 4704 of 512 96 | 92.4 (3), 9800 124.5 | 117 (5), 19600 184.5 | 177 (7), 12544
// of 384 113 | 109.4 (7).  Down to two thirds of that where the workgroups, with the input side at half of the rows live, are then two a unit and no
// more, so that none starts late: 9408 rows of 768 in two | three chunks 161.6 | 169.8, 15680 of 512 in four | five | six 151.0 | 154.7 | 152.8, 11956 of
// 448 in five, the wide side's in six 119.5 | 124.6.  Few chunks are long chains of products into one sum: relative error of dW (2-norm, to 64 bits), 2548 rows of 1024
// columns in one chunk 3.05e-7 as one sum, 1.06e-7 as sums of 256 rows (in four chunks 1.12e-7), 9800 of 512 in seven 2.26e-7, 1.11e-7 (in ten
// and sixteen 1.60e-7); 1 us of a step of 103 to 150.
// The narrow side is a chain of steps on few units where it is called alone, so its chunks are of about 1325 live rows at most where that
// is a good deal fewer.  With the input side and the wide side they are then two workgroups a unit, or else many and short, behind
// the others.  As many chunks as the wide side's | so, us, called alone (as many as fill the chip) and a step: 5096 rows of 1024 columns 29.7 | 24.2
// (26.8) and 147.0 | 147.7, 6664 26.1 | 24.2 (24.2), 180.5 | 178.2, 7056 of 832 26.5 | 21.1 (23.0), 160.0 | 154.4, 9408 of 768 31.3 | 21.8 (23.5),
// 160.6 | 162.4, 10976 27.0 | 22.2 (22.1), 177.1 | 179.4; not 9800 of 640 25.0 | 21.3 (24.2), 140.4 | 144.7.
inline int block_splits(int M_cap, int C, int N_out) {
  const long narrow = gemm_tiles<long>(C, C, kWeightEdge), wide = gemm_tiles<long>(3L * C, C, kWeightEdge);
  const long left = 512 - gemm_tiles<long>(std::max(M_cap / 2, 1), C, kWeightEdge), beside = left / (narrow + wide);
  long best = std::max((long)(std::sqrt(700. * M_cap) / C), 1L);
  if (beside < best && 3 * beside >= 2 * best) best = beside;
  if (N_out == C && M_cap > 3300 * best) {
    long more = (M_cap + 1325L) / 2650;
    if (more * narrow + best * wide > left) more = std::max(more, std::min(3 * best, 256 / narrow));
    best = std::max(best, std::min(more, weight_most_splits(M_cap, C, N_out, 0) - 1L));      // (fewer: the sums stay apart)
  }
  return (int)std::clamp(best, 1L, (long)weight_splits(M_cap, C, N_out, 0));
}
// The shape of a call of its own, by what was measured (half of the capacity live): a step takes
// 1.1 us in a round of two 128 x 128 workgroups a unit and 1.8 in one of 256 x 256 tiles, launch, first loads and last stores 6
// and 9 us, and the sums 0.15 us a MB of partial tiles.  cfg 2 | 8 forces the tiles (where they cannot add up sums apart, with the chunks that
// need no such sums).
inline WeightShape weight_shape(int M_cap, int K, int N_out, int cfg, int forced) {
  WeightShape small = {kWeightEdge, weight_most_splits(M_cap, K, N_out, forced)};
  WeightShape big = {256, weight_splits_big(M_cap, gemm_tiles<long>(N_out, K, 256), 16, forced)};
  if (of_a_block(K, N_out)) {
    if (forced <= 0 && cfg != 8 && in_one_launch(M_cap, K)) {
      const int few = block_splits(M_cap, K, N_out);
      if (few < small.splits) return {kWeightEdge, few, true};
    }
    big.splits = small.splits;
  }
  const double mb = 4e-6 * N_out * K;
  const auto steps = [&](int splits) { return (double)((std::max(M_cap / 2, 1) / splits + 63) / 64); };
  const double t_small = 6 + 1.1 * steps(small.splits) * std::ceil(small.splits * small.tiles(N_out, K) / 512.) + 0.15 * mb * small.splits;
  const double t_big = 9 + 1.8 * steps(big.splits) * std::ceil(big.splits * big.tiles(N_out, K) / 256.) + 0.15 * mb * big.splits;
  WeightShape shape = t_big < 0.97 * t_small ? big : small;
  if (cfg == 2 || cfg == 8) shape.edge = cfg == 8 ? 256 : kWeightEdge;
  return shape;
}

}  // namespace spa
