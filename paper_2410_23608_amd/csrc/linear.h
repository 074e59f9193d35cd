// Arguments of the row GEMM shared by the projections and the input side of their backward (linear.hip).
#pragma once

#include "gemm_shape.h"
#include "spa_common.h"

namespace spa {

struct GemmArgs {
  const __bf16* a;               // row a_idx[j] (or j), stride lda
  const int32_t* a_idx;
  long lda;
  const float* scores;           // kScale: row j of the product is multiplied by sigmoid(scores[a_idx[j]])
  const int32_t* total;          // live rows on the device, or null (m_cap)
  int m_cap, kc, ncols;
  const __bf16* w;
  const __bf16* bias;
  __bf16* out;                   // row o_idx[j] (or j), stride ldo; residual: same layout
  long ldo;
  const int32_t* o_idx;
  const __bf16* residual;
  const int32_t* inv_pos;        // given: the rows i < zrows of out with inv_pos[i] < 0 are zeroed (copied from residual)
  long zrows;
  LargeRule rule;                // of the large tiles (set by the launch)
};

// deep = false: out = A W^T (W [ncols][kc]); true: out = A W (W [kc][ncols]).
int launch_gemm_rows(const char* fn, const GemmArgs& args, bool deep, hipStream_t st);
// Inside a launch group (linear_bwd.hip): the row GEMM of a backward input side is noted; big: with large tiles.
int group_note_rows(const char* fn, const GemmArgs& args, bool big);

}  // namespace spa
