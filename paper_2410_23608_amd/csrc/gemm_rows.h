// The row GEMM of the projections and of the input side of their backward: out rows = rows of A times W^T or W.
#pragma once

#include <type_traits>

#include "gemm_async.h"
#include "linear.h"
#include "spa_common.h"

namespace spa {

// Workgroup tile BM x BN, WGM x WGN waves, each wave (BM / WGM) x (BN / WGN) of the output.
// kDeep = false: out = A W^T, W [ncols][kc] (forward); kDeep = true: out = A W, W [kc][ncols] (input side
// of the backward).  Either way the contraction has kc elements and runs along the rows of A.
template <bool kScale, bool kDeep, int BM, int BN, int WGM, int WGN, int STAGES>
__device__ __forceinline__ void gemm_rows_block(const GemmArgs& p, unsigned char* gemm_smem, unsigned block, unsigned blocks) {
  constexpr int THREADS = 64 * WGM * WGN, TM = BM / WGM / 32, TN = BN / WGN / 32;
  using PA = RowsPieces<BM, THREADS>;
  using PB = typename std::conditional<kDeep, DeepPieces<BN, THREADS>, RowsPieces<BN, THREADS>>::type;
  __bf16* lds = reinterpret_cast<__bf16*>(gemm_smem);
  __shared__ float bias_s[BN];     // bias of the tile's output columns (0 past the edge or without bias)
  __shared__ int o_row[BM];        // output row of every tile row

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
  // Tile order.  Workgroup ids go to the 8 XCDs round-robin (id % 8) and each XCD has its own
  // L2.  The LIVE tiles (the row count is only known here, on the device) are numbered m-major
  // and cut into 8 equal contiguous ranges, one per XCD: the workgroups that share a block of A
  // rows run on one XCD, and every XCD gets the same number of tiles.
  const int M = p.total != nullptr ? min(p.total[0], p.m_cap) : p.m_cap;
  const int live_tiles = ((M + BM - 1) / BM) * p.n_tiles, per_xcd = (live_tiles + 7) >> 3;
  const int xcd = block & 7, jx = block >> 3, tile_id = xcd * per_xcd + jx;
  if (jx < per_xcd && tile_id < live_tiles) {
    const int mt = tile_id / p.n_tiles, nt = tile_id - mt * p.n_tiles;
    const int m0 = mt * BM, n0 = nt * BN;
    const int wm = (wv / WGN) * TM * 32, wn = (wv % WGN) * TN * 32;

    // rows past the end fetch the last valid row and columns past the edge a valid column: they only
    // reach outputs that are never stored
    const __bf16* ap[PA::kCount];
    const __bf16* bp[PB::kCount];
    const int a_col = PA::col(tid), b_col = PB::col(tid);
#pragma unroll
    for (int u = 0; u < PA::kCount; ++u) {
      const int r = min(m0 + PA::row0(tid) + u * PA::kRowStep, M - 1);
      ap[u] = p.a + (p.a_idx != nullptr ? (long)p.a_idx[r] : (long)r) * p.lda + a_col;
    }
    float row_scale[TM];
    if (kScale) {
#pragma unroll
      for (int i = 0; i < TM; ++i) row_scale[i] = p.scores[p.a_idx[min(m0 + wm + i * 32 + l32, M - 1)]];
    }
#pragma unroll
    for (int u = 0; u < PB::kCount; ++u) {
      const int r = PB::row0(tid) + u * PB::kRowStep;
      bp[u] = kDeep ? p.w + (long)r * p.ncols + (n0 + b_col < p.ncols ? n0 + b_col : n0)
                    : p.w + (long)min(n0 + r, p.ncols - 1) * p.kc + b_col;
    }
    for (int t = tid; t < BN; t += THREADS)
      bias_s[t] = p.bias != nullptr && n0 + t < p.ncols ? static_cast<float>(p.bias[n0 + t]) : 0.f;
    for (int t = tid; t < BM; t += THREADS) o_row[t] = p.o_idx != nullptr && m0 + t < M ? p.o_idx[m0 + t] : m0 + t;

    const int nk = (p.kc + kGaK - 1) / kGaK, k_tail = p.kc % kGaK;
    const __bf16* zeros = reinterpret_cast<const __bf16*>(gemm_zeros);
    const long b_step = kDeep ? (long)kGaK * p.ncols : kGaK;
    // the last step may be partial: pieces past the contraction are zero in both operands
    auto next_a = [&](int u, int t) {
      const __bf16* g = ap[u];
      ap[u] += kGaK;
      if (k_tail != 0 && t == nk - 1 && a_col >= k_tail) g = zeros;
      return g;
    };
    auto next_b = [&](int u, int t) {
      const __bf16* g = bp[u];
      bp[u] += b_step;
      if (k_tail != 0 && t == nk - 1 && (kDeep ? PB::row0(tid) + u * PB::kRowStep : b_col) >= k_tail) g = zeros;
      return g;
    };
    auto frag_a = [&](const __bf16* tile, int i, int kk) { return rows_frag(tile, wm + i * 32, kk, l32, hh); };
    auto frag_b = [&](const __bf16* tile, int j, int kk) {
      if constexpr (kDeep) return deep_frag<BN>(tile, kk, wn + j * 32, lane);
      else return rows_frag(tile, wn + j * 32, kk, l32, hh);
    };
    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    gemm_async_loop<BM * kGaK, BN * kGaK, PA::kCount, PB::kCount, STAGES, THREADS, TM, TN>(lds, nk, next_a, next_b, frag_a,
                                                                                           frag_b, acc);

    // epilogue: scale, bias, bf16; 32 rows of the wave at a time are parked in its own part of LDS (LDS
    // operations of a wave complete in order) and leave as whole 16-byte pieces.  The pieces of the residual are
    // fetched together, pieces past the edge from a valid place (one at a time where they are added, each waits
    // for memory: the output projection of 64 x 196 tokens of 384 columns 11.4 -> 9.8 us)
    constexpr int NC = TN * 32, ORS = NC + 8, PIECES = NC / 8, PER_LANE = 32 * PIECES / 64;
    static_assert(WGM * WGN * 2 * 32 * ORS <= STAGES * (BM + BN) * kGaK, "output staging fits in the operand buffers");
    auto epilogue = [&](auto with_residual) {
      constexpr bool kResidual = decltype(with_residual)::value;
      bf16x8 res[kResidual ? TM : 1][kResidual ? PER_LANE : 1];
      if constexpr (kResidual) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int u = 0; u < PER_LANE; ++u) {
            const int c = lane + 64 * u, row = min(wm + i * 32 + c / PIECES, M - 1 - m0), n = n0 + wn + c % PIECES * 8;
            res[i][u] = *reinterpret_cast<const bf16x8*>(p.residual + (long)o_row[row] * p.ldo + (n < p.ncols ? n : n0));
          }
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        __bf16* tile = lds + (wv * 2 + (i & 1)) * 32 * ORS;
        const float rs = kScale ? sigmoidf_dev(row_scale[i]) : 1.f;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int n = j * 32 + 8 * g + 4 * hh;        // 4 consecutive output columns
            floatx4 f = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
            if (kScale) f *= rs;
            f += *reinterpret_cast<const floatx4*>(&bias_s[wn + n]);
            *reinterpret_cast<bf16x4*>(&tile[l32 * ORS + n]) = __builtin_convertvector(f, bf16x4);
          }
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u) {
          const int c = lane + 64 * u, r = c / PIECES, ch = c % PIECES, row = wm + i * 32 + r, n = n0 + wn + ch * 8;
          bf16x8 val = *reinterpret_cast<const bf16x8*>(&tile[r * ORS + ch * 8]);
          if constexpr (kResidual) val = float_to_bf16x8(bf16x8_to_float(val) + bf16x8_to_float(res[i][u]));
          if (m0 + row < M && n < p.ncols) *reinterpret_cast<bf16x8*>(p.out + (long)o_row[row] * p.ldo + n) = val;
        }
      }
    };
    if (p.residual != nullptr) epilogue(std::true_type{});
    else epilogue(std::false_type{});
  }
  // The rows no packed row maps to: shared by the waves of the workgroups without a tile, which run beside
  // the others, or by all when those are few.
  if (p.inv_pos != nullptr) {
    constexpr int NW = WGM * WGN;
    const int live = min((int)blocks, 8 * per_xcd), idle = (int)blocks - live;
    const bool by_idle = 4 * idle >= live;
    const long units = (long)(by_idle ? idle : (int)blocks) * NW;
    const long u = ((long)block - (by_idle ? live : 0)) * NW + wv;      // (idle: jx >= per_xcd, i.e. block >= 8 per_xcd)
    if (u < 0) return;
    const long per = (p.zrows + units - 1) / units, r0 = min(p.zrows, u * per), r1 = min(p.zrows, r0 + per);
    zero_unselected_rows(p.out, p.ldo, p.ncols, p.inv_pos, r0, r1, lane, p.residual);
  }
}

template <bool kScale, bool kDeep, int BM, int BN, int WGM, int WGN, int STAGES>
__global__ void __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(BM > 128 ? 1 : 2)))
gemm_rows_kernel(const GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_smem[];
  gemm_rows_block<kScale, kDeep, BM, BN, WGM, WGN, STAGES>(p, gemm_smem, blockIdx.x, gridDim.x);
}

}  // namespace spa
