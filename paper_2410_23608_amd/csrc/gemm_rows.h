// The row GEMM of the projections and of the input side of their backward: out rows = rows of A times W^T or W.
#pragma once

#include <type_traits>

#include "gemm_async.h"
#include "gemm_shape.h"
#include "linear.h"
#include "spa_common.h"

namespace spa {

// Workgroup tile BM x BN, WGM x WGN waves, each wave (BM / WGM) x (BN / WGN) of the output.
// kDeep = false: out = A W^T, W [ncols][kc] (forward); kDeep = true: out = A W, W [kc][ncols] (input side
// of the backward).  Either way the contraction has kc elements and runs along the rows of A.
// The rows [m_first, M) of the output; returns how many workgroups have a tile.
template <class MF, bool kScale, bool kDeep, bool LOOP, int BM, int BN, int WGM, int WGN, int SA, int SB>
__device__ __forceinline__ int gemm_rows_tiles(const GemmArgs& p, unsigned char* gemm_smem, unsigned block, unsigned blocks,
                                               int m_first, int M) {
  constexpr int E = MF::kEdge, THREADS = 64 * WGM * WGN, TM = BM / WGM / E, TN = BN / WGN / E;
  static_assert(BM == WGM * TM * E && BN == WGN * TN * E, "whole matrix tiles");
  using PA = RowsPieces<MF, BM, THREADS>;
  using PB = typename std::conditional<!kDeep, RowsPieces<MF, BN, THREADS>,
                                      typename std::conditional<E == 16, DeepBlocks<BN, THREADS>, DeepPieces<BN, THREADS>>::type>::type;
  __bf16* lds = reinterpret_cast<__bf16*>(gemm_smem);
  constexpr int NC = TN * E, ORS = NC + 8, PIECES = NC / 8, PER_LANE = E * PIECES / 64, STAGING = WGM * WGN * 2 * E * ORS;
  __shared__ float bias_s[BN];     // bias of the tile's output columns (0 past the edge or without bias)
  __shared__ int o_row[BM];        // output row of every tile row
  static_assert(E * PIECES % 64 == 0 && STAGING <= (SA * BM + SB * BN) * kGaK, "output staging fits in the operand buffers");

  // Tile order.  Workgroup ids go to the 8 XCDs round-robin (id % 8) and each XCD has its own
  // L2.  The LIVE tiles (the row count is only known here, on the device) are numbered m-major
  // and cut into 8 equal contiguous ranges, one per XCD: the workgroups that share a block of A
  // rows run on one XCD, and every XCD gets the same number of tiles.
  const int n_tiles = (p.ncols + BN - 1) / BN, live_tiles = ((M - m_first + BM - 1) / BM) * n_tiles, per_xcd = (live_tiles + 7) >> 3;
  // A workgroup takes the tiles jx, jx + blocks / 8, ... of its XCD's range.
  const int xcd = block & 7;
  for (int jx = block >> 3; jx < per_xcd && xcd * per_xcd + jx < live_tiles; jx += blocks >> 3) {
    const int tid = LOOP ? fresh_thread_id() : threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), tile_id = xcd * per_xcd + jx;
    const int mt = tile_id / n_tiles, nt = tile_id - mt * n_tiles;
    const int m0 = m_first + mt * BM, n0 = nt * BN;
    const int wm = (wv / WGN) * TM * E, wn = (wv % WGN) * TN * E;

    // rows past the end fetch the last valid row and columns past the edge a valid column: they only
    // reach outputs that are never stored
    const __bf16* ap[PA::kCount];
    const __bf16* bp[PB::kCount];
    const int a_col = PA::col(tid, 0);
    int a_row[PA::kCount];
#pragma unroll
    for (int u = 0; u < PA::kCount; ++u) a_row[u] = min(m0 + PA::row(tid, u), M - 1);
    if (p.a_idx != nullptr) {
#pragma unroll
      for (int u = 0; u < PA::kCount; ++u) a_row[u] = p.a_idx[a_row[u]];
    }
    // bias and output row of the thread's column and row; they go to the tables when the products are done
    static_assert(BM <= THREADS && BN <= THREADS, "one of each a thread");
    __bf16 bias_v = static_cast<__bf16>(0.f);
    int o_v = m0 + tid;
    if (p.bias != nullptr && tid < BN && n0 + tid < p.ncols) bias_v = p.bias[n0 + tid];
    if (p.o_idx != nullptr && tid < BM && m0 + tid < M) o_v = p.o_idx[m0 + tid];
#pragma unroll
    for (int u = 0; u < PA::kCount; ++u) ap[u] = p.a + (long)a_row[u] * p.lda + a_col;
    float row_scale[TM];
    if (kScale) {
#pragma unroll
      for (int i = 0; i < TM; ++i) row_scale[i] = p.scores[p.a_idx[min(m0 + wm + i * E + lane % E, M - 1)]];
    }
#pragma unroll
    for (int u = 0; u < PB::kCount; ++u) {
      const int r = PB::row(tid, u), b_col = PB::col(tid, u);
      bp[u] = kDeep ? p.w + (long)r * p.ncols + (n0 + b_col < p.ncols ? n0 + b_col : n0)
                    : p.w + (long)min(n0 + r, p.ncols - 1) * p.kc + b_col;
    }
    const int nk = (p.kc + kGaK - 1) / kGaK, k_tail = p.kc % kGaK;
    const __bf16* zeros = reinterpret_cast<const __bf16*>(gemm_zeros);
    const long b_step = kDeep ? (long)kGaK * p.ncols : kGaK;
    // the last step may be partial: pieces past the contraction are zero in both operands
    auto next_a = [&](int u, int t, auto inside) {
      const __bf16* g = ap[u];
      ap[u] += kGaK;
      if (!inside && k_tail != 0 && t == nk - 1 && a_col >= k_tail) g = zeros;
      return g;
    };
    auto next_b = [&](int u, int t, auto inside) {
      const __bf16* g = bp[u];
      bp[u] += b_step;
      if (!inside && k_tail != 0 && t == nk - 1 && (kDeep ? PB::row(tid, u) : PB::col(tid, u)) >= k_tail) g = zeros;
      return g;
    };
    auto frag_a = [&](const __bf16* tile, int i, int kk) { return rows_frag<MF>(tile, wm + i * E, kk, lane); };
    auto frag_b = [&](const __bf16* tile, int j, int kk) {
      if constexpr (kDeep && E == 16) return deep_block_frag(tile, kk, wn + j * E, lane);
      else if constexpr (kDeep) return deep_frag<BN>(tile, kk, wn + j * E, lane);
      else return rows_frag<MF>(tile, wn + j * E, kk, lane);
    };
    auto tables = [&] {
      if (tid < BN) bias_s[tid] = static_cast<float>(bias_v);
      if (tid < BM) o_row[tid] = o_v;
    };
    typename MF::Acc acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 4 * MF::kGroups; ++r) acc[i][j][r] = 0.f;
    gemm_async_loop<MF, BM * kGaK, BN * kGaK, PA::kCount, PB::kCount, SA, SB, THREADS, TM, TN>(lds, nk, next_a, next_b, frag_a,
                                                                                               frag_b, acc, tables);

    // epilogue: scale, bias, bf16; the EDGE rows of a row of matrix tiles at a time are parked in its own part of LDS (LDS
    // operations of a wave complete in order) and leave as whole 16-byte pieces.  The pieces of the residual of the
    // next row of tiles are fetched while this one is added and stored, pieces past the edge from a valid place (one at a
    // time where they are added, each waits for memory: the output projection of 64 x 196 tokens of 384 columns 11.4 -> 9.8 us;
    // all together they are 64 registers beside the 128 accumulators of 256 x 256 tiles, and spill).
    auto epilogue = [&](auto with_residual) {
      constexpr bool kResidual = decltype(with_residual)::value;
      bf16x8 res[2][kResidual ? PER_LANE : 1];
      auto fetch = [&](int i) {
        if constexpr (kResidual) {
#pragma unroll
          for (int u = 0; u < PER_LANE; ++u) {
            const int c = lane + 64 * u, row = min(wm + i * E + c / PIECES, M - 1 - m0), n = n0 + wn + c % PIECES * 8;
            res[i & 1][u] = *reinterpret_cast<const bf16x8*>(p.residual + (long)o_row[row] * p.ldo + (n < p.ncols ? n : n0));
          }
        }
      };
      fetch(0);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        __bf16* tile = lds + (wv * 2 + (i & 1)) * E * ORS;
        const float rs = kScale ? sigmoidf_dev(row_scale[i]) : 1.f;
        if (i + 1 < TM) fetch(i + 1);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int g = 0; g < MF::kGroups; ++g) {
            const int n = j * E + MF::row(g, lane);       // 4 consecutive output columns
            floatx4 f = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
            if (kScale) f *= rs;
            f += *reinterpret_cast<const floatx4*>(&bias_s[wn + n]);
            *reinterpret_cast<bf16x4*>(&tile[lane % E * ORS + n]) = __builtin_convertvector(f, bf16x4);
          }
        if (kResidual) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < PER_LANE; ++u) {
          const int c = lane + 64 * u, r = c / PIECES, ch = c % PIECES, row = wm + i * E + r, n = n0 + wn + ch * 8;
          bf16x8 val = *reinterpret_cast<const bf16x8*>(&tile[r * ORS + ch * 8]);
          if constexpr (kResidual) val = float_to_bf16x8(bf16x8_to_float(val) + bf16x8_to_float(res[i & 1][u]));
          if (m0 + row < M && n < p.ncols) *reinterpret_cast<bf16x8*>(p.out + (long)o_row[row] * p.ldo + n) = val;
        }
        if (kResidual) __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (p.residual != nullptr) epilogue(std::true_type{});
    else epilogue(std::false_type{});
    if (!LOOP) break;
    __syncthreads();                 // the tables and buffers are read to the end
  }
  return min((int)blocks, 8 * per_xcd);
}
// The rows no packed row maps to.  The waves of the workgroups without a tile (from the live-th on) take as many as they clear or
// copy while the others multiply; what is left is shared by all.
__device__ __forceinline__ void gemm_unmapped_rows(const GemmArgs& p, int M, unsigned block, unsigned blocks, int live, int waves) {
  if (p.inv_pos == nullptr) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const long all = p.zrows, idle = (long)((int)blocks - live) * waves, busy = (long)live * waves;
  const float spread = (float)all / (float)max(all - M, 1L);          // rows of out for one without a packed row
  const long alone = (long)min(p.rule.fit * spread + 1.f, (float)all);    // rows of out for a wave without a tile, while the others multiply
  const long rest = max(0L, all - idle * alone), share = rest > 0 ? (rest + idle + busy - 1) / (idle + busy) : 0;
  const long per_idle = rest > 0 ? alone + share : idle > 0 ? (all + idle - 1) / idle : 0;
  const long u = (long)((int)block - live) * waves + wv;              // (below 0: with a tile, counted from the first)
  const long r0 = u >= 0 ? u * per_idle : idle * per_idle + (u + busy) * share, r1 = r0 + (u >= 0 ? per_idle : share);
  zero_unselected_rows<4, 2>(p.out, p.ldo, p.ncols, p.inv_pos, min(r0, all), min(r1, all), lane, p.residual);
}
__device__ __forceinline__ int gemm_live_rows(const GemmArgs& p) { return p.total != nullptr ? min(p.total[0], p.m_cap) : p.m_cap; }
// 128 x 128 tiles, a workgroup each.  The rows no packed row maps to: shared by the waves of the workgroups without a tile, or by all
// when those are few.
template <bool kScale, bool kDeep, int STEPS, int THREADS>
__device__ __forceinline__ void gemm_rows_small(const GemmArgs& p, unsigned char* gemm_smem, unsigned block, unsigned blocks) {
  constexpr int NW = THREADS / 64;
  const int live = gemm_rows_tiles<Mfma32, kScale, kDeep, false, 128, 128, 2, NW / 2, STEPS, STEPS>(p, gemm_smem, block, blocks, 0, gemm_live_rows(p));
  if (p.inv_pos == nullptr) return;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, idle = (int)blocks - live;
  const bool by_idle = 4 * idle >= live;
  const long units = (long)(by_idle ? idle : (int)blocks) * NW;
  const long u = ((long)block - (by_idle ? live : 0)) * NW + wv;      // (idle: jx >= per_xcd, i.e. block >= live)
  if (u < 0) return;
  const long per = (p.zrows + units - 1) / units, r0 = min(p.zrows, u * per), r1 = min(p.zrows, r0 + per);
  zero_unselected_rows(p.out, p.ldo, p.ncols, p.inv_pos, r0, r1, lane, p.residual);
}

constexpr size_t kGemmSmallLds = (size_t)2 * (128 + 128) * kGaK * sizeof(__bf16), kGemmRingLds = 2 * kGemmSmallLds;
// steps of A and of B in LDS: three of 192 + 192, three of 256 and two of 192, two of 256 + 256
constexpr size_t kGemmBigLds = (size_t)std::max({3 * 192 + 3 * 192, 3 * 256 + 2 * 192, 2 * 256 + 2 * 256}) * kGaK * sizeof(__bf16);

// 128 x 128 tiles: four waves of 64 x 64, two workgroups per unit.
template <bool kScale, bool kDeep>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) gemm_rows_small_kernel(const GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_smem[];
  gemm_rows_small<kScale, kDeep, 2, 256>(p, gemm_smem, blockIdx.x, gridDim.x);
}
// 128 x 128 tiles where a unit has one: eight waves of 64 x 32 and four steps of both operands in LDS.  With four waves and two steps
// a wave alone on its SIMD issues loads, reads and products one after the other (0.6 us a step; the products alone 0.2) and a
// step's loads have one step to come; now 0.37 us.  us, called again and again, before -> now (four waves with four steps): 1568 rows
// of 2304 -> 768 25.0 -> 17.3 (20.6; loads dealt out 18.2), 784 of 3072 -> 1024 34.0 -> 21.5 (26.3; 22.5), 2000 of 1024 -> 1024 12.3 ->
// 10.2 (11.6; 10.9), 6272 of 1152 -> 384 13.9 -> 10.9, 6272 of 384 -> 384 with the residual 8.9 -> 8.2, 98 rows 7.1 -> 6.4.  Resident
// workgroups that walk the tiles take 0.5 us more.
template <bool kScale, bool kDeep>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) gemm_rows_ring_kernel(const GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_smem[];
  gemm_rows_small<kScale, kDeep, 4, 512>(p, gemm_smem, blockIdx.x, gridDim.x);
}

// The same waves with two steps in LDS, two workgroups a unit (two_rings of gemm_shape.h).
template <bool kScale, bool kDeep>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) gemm_rows_eight_kernel(const GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_smem[];
  gemm_rows_small<kScale, kDeep, 2, 512>(p, gemm_smem, blockIdx.x, gridDim.x);
}

// Tiles of 256 x 256 (eight waves of 128 x 64), 256 x 192 (eight of 64 x 96) or 192 x 192 (eight of 48 x 96); the fewer accumulators and
// columns of the latter two leave LDS for a third step of the rows of A, or of both: a step of K 2304 waits for rows that no other
// unit has fetched yet, and with two steps its loads have one step to come (256 x 192 with two steps of both 63.7 us, with three of
// A 53).  One resident workgroup per unit walks the tiles (a workgroup per tile of the capacity: 1.5 us more for those without
// one), and the rounds that takes decide (large_plan); the row count is only known here.  Measured, called again and again, random
// operands, 192 x 192 | 256 x 192 | 256 x 256, rounds in brackets, us: K 768, 11540 rows of 768 columns 18.4 (1) | 20.6 (1) |
// 21.5 (1), 13500 rows 30.3 (2) | 21.2 (1) | 22.0 (1); rows of 2304 columns: 7526 31.7 (2) | 36.8 (2) | 43.5 (2), 11540 47.9 (3) |
// 55 (3) | 46 (2), 12544 61 (4) | 58 (3) | 51 (2), the first 7168 rows of them 256 x 256 and the others 256 x 192 47.4, 15052 66 (4) |
// 63.5 (3) | 71 (3); K 2304, rows of 768 columns: 11540 47 (1) | 51 (1) | 60 (1), 12544 77 (2) | 52.8 (1) | 61 (1).  No unit is busy
// for much more than a third of a launch (matrix pipe 35 %, LDS 19 %, address units 34 % of QKV's with both shapes; the L2 delivers
// 11 TB/s in the loop, 6.5 over the launch): what binds is the order within a step, wait, barrier, loads, products, with one
// workgroup a unit to fill the gaps.  Four waves of 128 x 128 (a third fewer LDS reads) took 56 us for 12544 rows of 2304 columns.
enum class Large { kByRows, k192, k256, k256x192 };        // kByRows: the plan for the live rows (gemm_shape.h)
template <bool kScale, bool kDeep, Large SHAPE>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(1))) gemm_rows_big_kernel(const GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char gemm_smem[];
  const unsigned block = blockIdx.x, blocks = gridDim.x;
  const int M = gemm_live_rows(p);
  LargePlan plan = {SHAPE == Large::k192, SHAPE == Large::k256 ? M : 0, 0, 0};
  if (SHAPE == Large::kByRows) plan = large_plan(M, p.ncols, p.inv_pos != nullptr ? (int)min(max(p.zrows - M, 0L), 2147483647L) : 0, p.rule);
  int live = 0;
  if (SHAPE == Large::k192 || (SHAPE == Large::kByRows && plan.medium)) {
    live = gemm_rows_tiles<Mfma16, kScale, kDeep, true, 192, 192, 4, 2, 3, 3>(p, gemm_smem, block, blocks, 0, M);
  } else {
    if (SHAPE != Large::k256x192 && plan.wide_rows > 0)
      live = gemm_rows_tiles<Mfma32, kScale, kDeep, true, 256, 256, 2, 4, 2, 2>(p, gemm_smem, block, blocks, 0, plan.wide_rows);
    if (SHAPE != Large::k256 && plan.wide_rows < M)
      live = max(live, gemm_rows_tiles<Mfma16, kScale, kDeep, true, 256, 192, 4, 2, 3, 2>(p, gemm_smem, block, blocks, plan.wide_rows, M));
  }
  gemm_unmapped_rows(p, M, block, blocks, live, 8);
}

}  // namespace spa
