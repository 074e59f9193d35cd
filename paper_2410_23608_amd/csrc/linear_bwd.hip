// Backward of the projections of the packed tokens (the 3 L C^2 and N C^2 terms of the SPA
// complexity formula, Section 3.2).  For out_j = r_j W^T + bias, with r_j the (gathered,
// optionally gate-scaled) row j and g_j the upstream gradient of out_j:
//   input side    d_rows[j,:] = g_j W                       [M, N_out] x [N_out, K]
//   weight side   dW = sum_j g_j^T r_j, dbias = sum_j g_j   [N_out, M] x [M, K]
// Both are MFMA GEMMs whose contraction index is the slow index of at least one operand in
// memory (W is [N_out][K] and the input side contracts over N_out; the weight side contracts
// over the tokens).  Those operands are staged in LDS exactly as they lie in memory, rows =
// contraction index, with whole 16-byte pieces, and the MFMA fragments are taken with the
// transposing LDS read (ds_read_b64_tr_b16), so nothing is transposed in memory or staged twice.
//
// Input side: the row GEMM of linear.hip, which also folds in the gather of the upstream rows (dout_idx),
// the scatter of the result rows (dx_idx) and the zero fill of the rows no packed row maps to.
// Weight side: the output is only N_out x K (a few dozen 128 x 128 tiles), so the tokens are
// cut into `splits` chunks (chunk length fixed on the device from the live row count, so all
// chunks carry work) and every (chunk, tile) is a workgroup; the partial tiles go to a
// workspace in fp32 and a second kernel adds them in chunk order: deterministic, no atomics.
// The operands come through the pipelined loop of gemm_async.h (weight_gemm_kernel); rows that have to be
// multiplied by the gate scale and rounded on the way cannot go straight to LDS and keep the kernel that
// stages them through registers (linear_bwd_weight_bf16_kernel).
// fp32 (tiny workload): one thread per output element.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "attn_tiles.h"
#include "gemm_async.h"
#include "gemm_rows.h"
#include "group.h"
#include "linear.h"
#include "spa_common.h"
#include "weight_shape.h"

namespace spa {

constexpr int kLbThreads = 256;
constexpr int kLbT = kWeightEdge;  // output tile edge
constexpr int kLbK = 64;           // contraction step
constexpr int kLbRS = kLbT + 16;   // row stride (elements) of a [contraction][128] tile: 72 dwords = 8 mod 64,
                                   // the 4 rows x 32 bytes a 16-lane block reads fall on distinct banks
constexpr int kLbRows = 512;       // rows of a chunk whose sources are tabled in LDS at a time (6 KB: with the
                                   // operand stages 78 KB per workgroup, two workgroups per compute unit)
constexpr size_t kLbGemmLds = (size_t)2 * 2 * kLbK * kLbT * sizeof(__bf16);   // two operand stages
constexpr size_t kLdsBytes = 160 * 1024;
constexpr size_t kLbWeightLds = (size_t)2 * 2 * kLbK * kLbRS * sizeof(__bf16);

// MFMA operand fragment taken DOWN the columns of a row-major tile whose rows are the
// contraction index: lane (l32, hh) receives tile[k0 + 8 hh + e][c0 + l32], e = 0..7, the same
// contraction order as a 16-byte read along a row of a [column][contraction] tile.  Within each
// block of 16 lanes the transposing read hands lane i, element e, the value that lane
// (4 e + i / 4) of the block addressed at its own element i % 4: lane s of a block points at
// row k0 + s / 4, columns 4 (s % 4) .. + 3, and lane i receives rows k0 .. k0 + 3 of column i.
template <int RS>
__device__ __forceinline__ bf16x8 frag_down_columns(const __bf16* tile, int k0, int c0, int lane) {
  const int blk = lane >> 4, s = lane & 15;
  const __bf16* p = tile + (k0 + 8 * (blk >> 1) + (s >> 2)) * RS + c0 + 16 * (blk & 1) + 4 * (s & 3);
  typedef shortx4_lds __attribute__((address_space(3))) * lds_ptr;
  const shortx4_lds lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
  const shortx4_lds hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * RS));
  const bf16x4 l4 = __builtin_bit_cast(bf16x4, lo), h4 = __builtin_bit_cast(bf16x4, hi);
  return __builtin_shufflevector(l4, h4, 0, 1, 2, 3, 4, 5, 6, 7);
}

// ------------------------------------------------------------------------------ input side (fp32)
__global__ void __launch_bounds__(256)
linear_bwd_input_f32_kernel(const float* __restrict__ dout, const int32_t* __restrict__ dout_idx, long ldd,
                            const int32_t* __restrict__ total, const float* __restrict__ W, int m_cap, int kc, int ncols,
                            float* __restrict__ dx, long ldx, const int32_t* __restrict__ dx_idx,
                            const int32_t* __restrict__ inv_pos, long rows) {
  const long stride = (long)gridDim.x * blockDim.x, first = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (inv_pos != nullptr)
    for (long i = first; i < rows * ncols; i += stride) {
      const long r = i / ncols;
      if (inv_pos[r] < 0) dx[r * ldx + (i - r * ncols)] = 0.f;
    }
  const int M = total != nullptr ? min(total[0], m_cap) : m_cap;
  for (long i = first; i < (long)M * ncols; i += stride) {
    const int m = (int)(i / ncols), c = (int)(i - (long)m * ncols);
    const float* g = dout + (dout_idx != nullptr ? (long)dout_idx[m] : (long)m) * ldd;
    float a = 0.f;
    for (int n = 0; n < kc; ++n) a = fmaf(g[n], W[(long)n * ncols + c], a);
    dx[(dx_idx != nullptr ? (long)dx_idx[m] : (long)m) * ldx + c] = a;
  }
}

// ----------------------------------------------------------------------------- weight side
// Chunk length and number of chunks that carry rows, from the live row count.
struct TokenSplit {
  int chunk, live;
};
__device__ __forceinline__ TokenSplit token_split(int M, int splits) {
  TokenSplit s;
  s.chunk = (((M + splits - 1) / splits) + kLbK - 1) & ~(kLbK - 1);
  s.live = s.chunk > 0 ? (M + s.chunk - 1) / s.chunk : 0;
  return s;
}

// The chunk of tokens and the tile of dW a workgroup takes.  Items are numbered chunk-major and cut into 8
// contiguous ranges, one per XCD, so the tiles that read the same rows share an L2.  At least one chunk
// (of no rows) exists: with no live rows the result is zero.
struct WeightItem {
  int split, n0, k0, m_begin, m_end;
  bool valid;
};
__device__ __forceinline__ WeightItem weight_item(int M, int splits, int n_tiles, int k_tiles, int live_min, int edge, unsigned block) {
  const TokenSplit ts = token_split(M, splits);
  const int tiles = n_tiles * k_tiles, items = max(ts.live, live_min) * tiles, per_xcd = (items + 7) >> 3;
  const int xcd = block & 7, jx = block >> 3, item = xcd * per_xcd + jx;
  WeightItem w = {};
  w.valid = jx < per_xcd && item < items;
  w.split = item / tiles;
  const int tile_id = item - w.split * tiles, nt = tile_id / k_tiles;
  w.n0 = nt * edge;
  w.k0 = (tile_id - nt * k_tiles) * edge;
  w.m_begin = w.split * ts.chunk;
  w.m_end = min(M, w.m_begin + ts.chunk);
  return w;
}

// 32 (n) x 64 (k) products of a wave leave as 16-byte pieces of 256-byte row segments through its own part of LDS (LDS
// operations of a wave complete in order); acc[j]: rows of the tile = k block j.
__device__ __forceinline__ void store_weight_block(const floatx16 (&acc)[2], float* tile, float* dst, int n_first, int k_first,
                                                   int n_out, int K, int lane) {
  constexpr int ORS = 64 + 4;
  const int l32 = lane & 31, hh = lane >> 5;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const floatx4 f = {acc[j][4 * g], acc[j][4 * g + 1], acc[j][4 * g + 2], acc[j][4 * g + 3]};
      *reinterpret_cast<floatx4*>(&tile[l32 * ORS + j * 32 + 8 * g + 4 * hh]) = f;
    }
#pragma unroll
  for (int c = lane; c < 32 * 16; c += 64) {
    const int r = c >> 4, ch = c & 15, n = n_first + r, k = k_first + ch * 4;
    if (n < n_out && k < K)
      *reinterpret_cast<floatx4*>(dst + (long)n * K + k) = *reinterpret_cast<const floatx4*>(&tile[r * ORS + ch * 4]);
  }
}

// part_w[split][n][k] = sum over the chunk's rows j of g_j[n] x_j[k]; part_b[split][n] = sum g_j[n] (from the fragments, in the
// workgroups of the first k tile).  Both operands have the contraction (the tokens) down their rows and come through the
// ring of gemm_async.h, rows of zeros past the chunk's end.  GI / XI: rows of g / x are named by an index array, read one
// step ahead of the loads that use it, without a branch (each branch made the compiler copy indices in flight, i.e. wait
// for them).  Tiles of 128 x 128 (four waves of 64 x 64, two workgroups a unit) or, EDGE 256, 256 x 256 (eight of 128 x 64).
// Addresses that step a pointer instead of a product and a select a load, and sums of the columns by vector additions,
// took a step of 128 x 128 tiles beside another workgroup from 1.35 to 1.06 us and one of 256 x 256 from 2.0 to 1.7.
// Measured with the sums, called again and again, 128 | 256, us: 12544 rows, 2304 x 768 in as many chunks as each fills the
// chip with 62 (72 before) | 58, 3072 x 1024 107 (132) | 86, 1536 x 512 35 | 38; gathered, 768 x 768 31.8 (36) | 37; 6272 rows,
// 2304 x 768 38.7 | 42.  In the chunks of a block's pair (weight_splits), by the rule, half of the rows live | all: 12544 rows,
// 2304 x 768 43 | 65, 768 x 768 24 | 33, 3072 x 1024 59 | 95, 1024 x 1024 30 | 47; 25088 rows, 768 x 768 34 | 61 (with the
// chunks of its own 33 | 49: the price of the same bits alone and in a group; the training steps run the pair).
struct WeightArgs {
  const __bf16* dout;
  const int32_t* dout_idx;
  long ldd;
  const __bf16* x;
  const int32_t *x_idx, *total;
  int m_cap, K, n_out, splits, n_tiles, k_tiles;
  bool fold;                     // the sums of every kFoldSteps steps are added up apart (128 x 128 tiles)
  float *part_w, *part_b;
};
constexpr int kFoldSteps = 4;    // (256 rows; WeightShape)
// TABLE: the indices of the chunk's named rows are in LDS, behind the operand stages, before the first step (a wait for an index from
// memory is one for every load issued before it, i.e. for all but one or two of the steps in flight).
template <int EDGE, int THREADS, int STAGES, bool TABLE, bool GI, bool XI>
__device__ __forceinline__ void weight_gemm_block(const WeightArgs& a, unsigned char* lb_smem, unsigned block) {
  constexpr int DEPTH = 64, WK = EDGE / 64, TM = EDGE * EDGE / (32 * THREADS);
  static_assert(TM <= WK && THREADS / 64 * TM * 32 * 64 == EDGE * EDGE, "a wave for the sums of every column block of g");
  using P = DeepPieces<EDGE, THREADS, DEPTH>;
  __bf16* lds = reinterpret_cast<__bf16*>(lb_smem);
  const long ldd = a.ldd;
  const int K = a.K, n_out = a.n_out;
  const int M = a.total != nullptr ? min(a.total[0], a.m_cap) : a.m_cap;
  const WeightItem w = weight_item(M, a.splits, a.n_tiles, a.k_tiles, 1, EDGE, block);
  if (!w.valid) return;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), wkb = wv % WK, wn = wv / WK * 32 * TM, wk = wkb * 64;
  const __bf16* zeros = reinterpret_cast<const __bf16*>(gemm_zeros);

  // columns past the matrix edge fetch a valid column (never stored)
  const int col = P::col(tid, 0), row = P::row(tid, 0);
  const __bf16* gcol = a.dout + (w.n0 + col < n_out ? w.n0 + col : w.n0);
  const __bf16* xcol = a.x + (w.k0 + col < K ? w.k0 + col : w.k0);
  const int rows = w.m_end - w.m_begin, nk = rows > 0 ? (rows + DEPTH - 1) / DEPTH : 0;
  // Named rows: their indices, those of the step to be issued next (past the end the last row's).  Rows in order: a
  // pointer to the thread's first.
  int gi[P::kCount], xi[P::kCount];
  constexpr bool kTable = TABLE && (GI || XI);
  int* g_table = reinterpret_cast<int*>(lb_smem + (size_t)STAGES * 2 * EDGE * DEPTH * sizeof(__bf16));
  int* x_table = g_table + (GI ? rows : 0);
  if (kTable) {
    for (int r = tid; r < rows; r += THREADS) {
      if (GI) g_table[r] = a.dout_idx[w.m_begin + r];
      if (XI) x_table[r] = a.x_idx[w.m_begin + r];
    }
    __syncthreads();
  }
  auto index = [&](int t) {
#pragma unroll
    for (int u = 0; u < P::kCount; ++u) {
      const int r = min(t * DEPTH + P::row(tid, u), rows - 1);
      if (GI) gi[u] = kTable ? g_table[r] : a.dout_idx[w.m_begin + r];
      if (XI) xi[u] = kTable ? x_table[r] : a.x_idx[w.m_begin + r];
    }
  };
  const __bf16* gp = gcol + (GI ? 0 : (long)(w.m_begin + row) * ldd);
  const __bf16* xp = xcol + (XI ? 0 : (long)(w.m_begin + row) * K);
  // the last step may be partial: rows past the end are zero in both operands
  const int tail = rows % DEPTH, partial = tail != 0 ? nk - 1 : -1;
  auto past = [&](int u, int t, const __bf16* p, auto inside) {
    if (!inside && t == partial) {
      asm volatile("" : "+v"(p));                    // (a branch: selects in every step cost more than it)
      p = P::row(tid, u) >= tail ? zeros : p;
    }
    return p;
  };
  auto next_g = [&](int u, int t, auto inside) {
    const __bf16* p = GI ? gcol + (size_t)(uint32_t)gi[u] * (size_t)ldd : gp;
    if (!GI) gp += (long)P::kRowStep * ldd;          // (a step's pieces are as far apart as the steps')
    return past(u, t, p, inside);
  };
  auto next_x = [&](int u, int t, auto inside) {
    const __bf16* p = XI ? xcol + (size_t)(uint32_t)xi[u] * K : xp;
    if (!XI) xp += (long)P::kRowStep * K;
    if ((GI || XI) && u == P::kCount - 1) index(t + 1);      // (the last address of step t has been formed)
    return past(u, t, p, inside);
  };
  static_assert(P::kCount * P::kRowStep == DEPTH, "pieces a constant distance apart");
  floatx16 acc[TM][2];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc[i][0][r] = 0.f;
      acc[i][1][r] = 0.f;
    }
  // Column block i of the wave's is number (i + wkb) % TM of g's, so that the first TM of the waves that hold the same blocks have
  // each another one as block 0, whose column sums it forms: of every 16 contraction elements a lane holds 8 of column l32.
  auto g_block = [&](int i) { return wn + (i + wkb) % TM * 32; };
  const bool do_bias = a.part_b != nullptr && w.k0 == 0 && wkb < TM;
  float colsum = 0.f;
  if ((GI || XI) && nk > 0) index(0);
  constexpr bool kFold = EDGE == kLbT;                      // (256 x 256 tiles have no registers for a second sum)
  floatx16 sum[kFold ? TM : 1][2];
#pragma unroll
  for (int i = 0; i < (kFold ? TM : 0); ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sum[i][0][r] = 0.f;
      sum[i][1][r] = 0.f;
    }
  auto fold = [&] {
#pragma unroll
    for (int i = 0; i < (kFold ? TM : 0); ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sum[i][j][r] += acc[i][j][r];
          acc[i][j][r] = 0.f;
        }
  };
  gemm_async_loop<Mfma32, EDGE * DEPTH, EDGE * DEPTH, P::kCount, P::kCount, STAGES, STAGES, THREADS, TM, 2, DEPTH>(
      lds, nk, next_g, next_x, [&](const __bf16* tile, int i, int kk) { return deep_frag<EDGE>(tile, kk, g_block(i), lane); },
      [&](const __bf16* tile, int j, int kk) { return deep_frag<EDGE>(tile, kk, wk + j * 32, lane); }, acc, [] {},
      [&](const bf16x8 (&g)[TM]) {
        if (do_bias) {
          const floatx8 f = bf16x8_to_float(g[0]);
          colsum += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
        }
      },
      [&](int t) {
        if (kFold && a.fold && (t + 1) % kFoldSteps == 0) fold();
      });
  fold();
  static_assert(THREADS / 64 * 32 * 68 * sizeof(float) <= STAGES * 2 * EDGE * DEPTH * sizeof(__bf16), "output staging fits in the operand stages");
  float* dst = a.part_w + (long)w.split * n_out * K;
#pragma unroll
  for (int i = 0; i < TM; ++i)
    store_weight_block(kFold ? sum[kFold ? i : 0] : acc[i], reinterpret_cast<float*>(lb_smem) + wv * 32 * 68, dst, w.n0 + g_block(i), w.k0 + wk, n_out, K, lane);
  if (do_bias) {
    const float s = sum_across_halves(colsum);
    const int n = w.n0 + g_block(0) + l32;
    if (hh == 0 && n < n_out) a.part_b[(long)w.split * n_out + n] = s;
  }
}
template <int EDGE, int THREADS>
__device__ __forceinline__ void weight_gemm_any(const WeightArgs& a, unsigned char* lb_smem, unsigned block) {
  const bool gi = a.dout_idx != nullptr, xi = a.x_idx != nullptr;
  if (!gi && !xi) weight_gemm_block<EDGE, THREADS, 2, false, false, false>(a, lb_smem, block);
  else if (!xi) weight_gemm_block<EDGE, THREADS, 2, false, true, false>(a, lb_smem, block);
  else if (!gi) weight_gemm_block<EDGE, THREADS, 2, false, false, true>(a, lb_smem, block);
  else weight_gemm_block<EDGE, THREADS, 2, false, true, true>(a, lb_smem, block);
}

constexpr size_t kLbBigLds = (size_t)2 * 2 * kLbK * 256 * sizeof(__bf16);
template <bool GI, bool XI>
__global__ void __launch_bounds__(kLbThreads) __attribute__((amdgpu_waves_per_eu(2))) weight_gemm_kernel(const WeightArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lb_smem[];
  weight_gemm_block<kLbT, kLbThreads, 2, false, GI, XI>(a, lb_smem, blockIdx.x);
}
// 128 x 128 tiles in eight waves of 32 x 64 with four steps of both operands in LDS, one workgroup a unit: the few chunks of a block's
// weight side where it is called alone, a chain of LDS reads and products at .55 us a step.  us a call with its sums, half of the rows live, two
// workgroups of four waves a unit | so: 768 x 768, 3136 rows 23.1 | 19.8, 6272 27.5 | 24.4; 1024 x 1024, 3136 rows 23.7 | 20.6; 512 x 512, 9800 rows
// 21.9 | 19.7; 3072 x 1024, 5096 rows 30.8 | 28.0; more tiles than units 2304 x 768, 11000 rows 38.7 | 44.9, 1536 x 512, 19600 rows 33.0 | 38.0.  Tiles
// of 128 x 64 in four waves 4 % faster where those are no more than units, 1 to 6 % slower where they are.
constexpr size_t kLbRingLds = 2 * kLbGemmLds;
template <bool GI, bool XI>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) weight_gemm_ring_kernel(const WeightArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lb_smem[];
  weight_gemm_block<kLbT, 512, 4, true, GI, XI>(a, lb_smem, blockIdx.x);
}
// Tiles of 256 x 256, eight waves, one workgroup a unit; up to two weight sides in a launch, workgroups [0, end) of the first.
struct WeightPair {
  WeightArgs w[2];
  unsigned end;
};
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(1))) weight_gemm_big_kernel(const WeightPair p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lb_smem[];
  const int s = blockIdx.x >= p.end;
  weight_gemm_any<256, 512>(p.w[s], lb_smem, blockIdx.x - (s ? p.end : 0u));
}

// A launch group of the projections' backward: an input side with 128 x 128 tiles and up to two weight sides in one
// launch (and the sums of both weight sides' chunks in one more).  On their own they leave units idle (98 rows, 384
// columns: 3 to 9 tiles) and wait for each other.  At 3136 rows of 384 columns the training step of a block takes
// 93 us so, 115 with the GEMMs one after the other and 110 with the weight sides on a second stream.  In eight waves a
// workgroup and a third step of A it was faster while the weight sides had 16 chunks (800 rows of 1024 columns 111 -> 102); with
// the chunks of block_splits, four | eight: 5096 rows of 1024 columns 145 | 148, 9408 of 768 159 | 161.5, 25088 of 128 92.3 | 94.3,
// 3920 of 192 62.2 | 61.4.
static_assert(kLbGemmLds == kGemmSmallLds, "the launch's LDS serves both");
struct LinearGroup {
  GemmArgs rows;
  WeightArgs w[2];
  unsigned end[2];               // workgroups of the input side, and of it and the first weight side
};
__global__ void __launch_bounds__(kLbThreads) __attribute__((amdgpu_waves_per_eu(2))) linear_bwd_group_kernel(const LinearGroup g) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lb_smem[];
  const unsigned block = blockIdx.x;
  if (block < g.end[0]) {
    gemm_rows_small<false, true, 2, 256>(g.rows, lb_smem, block, g.end[0]);
    return;
  }
  const int s = block >= g.end[1];
  const WeightArgs& a = g.w[s];
  weight_gemm_any<kLbT, kLbThreads>(a, lb_smem, block - g.end[s]);
}

// part_w[split][n][k] = sum over the chunk's rows j of g_j[n] r_j[k]; part_b[split][n] = sum g_j[n]
__global__ void __launch_bounds__(kLbThreads)
linear_bwd_weight_bf16_kernel(const __bf16* __restrict__ dout, const int32_t* __restrict__ dout_idx, long ldd,
                              const __bf16* __restrict__ x, const int32_t* __restrict__ x_idx,
                              const float* __restrict__ gate_scores, const int32_t* __restrict__ total, int m_cap, int K,
                              int n_out, int splits, int n_tiles, int k_tiles, float* __restrict__ part_w,
                              float* __restrict__ part_b) {
  constexpr int BT = kLbT, BK = kLbK, RS = kLbRS;
  extern __shared__ __attribute__((aligned(16))) unsigned char lb_smem[];
  __bf16(*Gs)[BK * RS] = reinterpret_cast<__bf16(*)[BK * RS]>(lb_smem);
  __bf16(*Xs)[BK * RS] = reinterpret_cast<__bf16(*)[BK * RS]>(lb_smem + 2 * BK * RS * sizeof(__bf16));
  __shared__ int g_src[kLbRows];       // row of dout (-1: past the end of the chunk), of x, and the
  __shared__ int x_src[kLbRows];       // gate scale of every row of the current block
  __shared__ float x_scale[kLbRows];

  const int M = total != nullptr ? min(total[0], m_cap) : m_cap;
  const TokenSplit ts = token_split(M, splits);
  const int tiles = n_tiles * k_tiles, items = ts.live * tiles, per_xcd = (items + 7) >> 3;
  const int xcd = blockIdx.x & 7, jx = blockIdx.x >> 3, item = xcd * per_xcd + jx;
  if (jx >= per_xcd || item >= items) return;
  const int split = item / tiles, tile_id = item - split * tiles;
  const int nt = tile_id / k_tiles, kt_ = tile_id - nt * k_tiles;
  const int n0 = nt * BT, k0 = kt_ * BT;
  const int m_begin = split * ts.chunk, m_end = min(M, m_begin + ts.chunk);

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
  const int wn = (wv >> 1) * 64, wk = (wv & 1) * 64;
  const bool do_bias = kt_ == 0 && wk == 0;

  // staging: both tiles are 64 token rows x 16 chunks of 16 bytes; thread -> chunk tid % 16 of
  // rows tid / 16 + 16 u.  Columns past the matrix edge load a valid column (never stored).
  constexpr int NU = 4;
  const int s_r = tid >> 4, s_c = tid & 15, lds_off = s_r * RS + s_c * 8;
  const __bf16* gcol = dout + (n0 + s_c * 8 < n_out ? n0 + s_c * 8 : n0);
  const __bf16* xcol = x + (k0 + s_c * 8 < K ? k0 + s_c * 8 : k0);

  struct Data {
    bf16x8 g[NU], x[NU];
    float sc[NU];
    bool ok[NU];
  };
  // rows of step t of the current block of tabled rows
  auto gload = [&](Data& d, int t) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int r = t * BK + s_r + u * 16;
      const int gi = g_src[r];
      d.ok[u] = gi >= 0;
      d.sc[u] = x_scale[r];
      d.g[u] = *reinterpret_cast<const bf16x8*>(gcol + (long)max(gi, 0) * ldd);
      d.x[u] = *reinterpret_cast<const bf16x8*>(xcol + (long)x_src[r] * K);
    }
  };
  auto lstore = [&](const Data& d, int buf) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      bf16x8 xv = d.x[u];
      xv = float_to_bf16x8(bf16x8_to_float(xv) * d.sc[u]);   // the gated row, rounded to bf16
      *reinterpret_cast<bf16x8*>(&Gs[buf][lds_off + u * 16 * RS]) = d.ok[u] ? d.g[u] : zero_bf16x8();
      *reinterpret_cast<bf16x8*>(&Xs[buf][lds_off + u * 16 * RS]) = d.ok[u] ? xv : zero_bf16x8();
    }
  };

  floatx16 acc[2][2], accb[2];
#pragma unroll
  for (int jn = 0; jn < 2; ++jn) {
#pragma unroll
    for (int r = 0; r < 16; ++r) accb[jn][r] = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][jn][r] = 0.f;
  }
  const __bf16 one = static_cast<__bf16>(1.0f);
  const bf16x8 ones = {one, one, one, one, one, one, one, one};

  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      bf16x8 xf[2], gf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) xf[i] = frag_down_columns<RS>(Xs[buf], kk * 16, wk + i * 32, lane);
#pragma unroll
      for (int jn = 0; jn < 2; ++jn) gf[jn] = frag_down_columns<RS>(Gs[buf], kk * 16, wn + jn * 32, lane);
      // tiles with rows = k (input feature), cols = n (output feature): a lane's 4 consecutive
      // accumulator registers are 4 consecutive k of one n, 16 bytes of a row of dW
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jn = 0; jn < 2; ++jn)
          acc[i][jn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[i], gf[jn], acc[i][jn], 0, 0, 0);
      if (do_bias) {
#pragma unroll
        for (int jn = 0; jn < 2; ++jn)
          accb[jn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, gf[jn], accb[jn], 0, 0, 0);
      }
    }
  };

  // The chunk is walked in blocks of kLbRows rows.  Where a block's rows lie (index arrays) and
  // their gate scale are tabled in LDS first, so the row loads of the pipelined loop depend on
  // LDS reads only, not on other loads still in flight (index -> score -> row would be three
  // dependent trips to memory per step).
  for (int blk0 = m_begin; blk0 < m_end; blk0 += kLbRows) {
    const int blk_rows = min(kLbRows, m_end - blk0), steps = (blk_rows + BK - 1) / BK;
    // all index loads first, then all score loads: two trips to memory for the whole table
    constexpr int NF = kLbRows / kLbThreads;
    int gi[NF], xi[NF];
    float sv[NF];
#pragma unroll
    for (int u = 0; u < NF; ++u) {
      const int m = min(blk0 + tid + u * kLbThreads, m_end - 1);
      gi[u] = dout_idx != nullptr ? dout_idx[m] : m;
      xi[u] = x_idx != nullptr ? x_idx[m] : m;
    }
#pragma unroll
    for (int u = 0; u < NF; ++u) sv[u] = gate_scores[xi[u]];
#pragma unroll
    for (int u = 0; u < NF; ++u) {
      const int r = tid + u * kLbThreads;
      const bool valid = r < blk_rows;
      if (r < steps * BK) {
        g_src[r] = valid ? gi[u] : -1;
        x_src[r] = valid ? xi[u] : 0;
        x_scale[r] = valid ? sigmoidf_dev(sv[u]) : 0.f;
      }
    }
    __syncthreads();
    // Entering a trip: LDS buffer 0 holds step kt, d1 holds step kt + 1, d0 is free.  Loads
    // past the last step repeat it; what they bring is stored but never multiplied.
    const int last = steps - 1;
    Data d0, d1;
    gload(d0, 0);
    if (steps > 1) gload(d1, 1);
    lstore(d0, 0);
    __syncthreads();
    for (int kt = 0; kt + 1 < steps; kt += 2) {
      gload(d0, min(kt + 2, last));
      compute(0);
      lstore(d1, 1);
      __syncthreads();
      gload(d1, min(kt + 3, last));
      compute(1);
      lstore(d0, 0);
      __syncthreads();
    }
    if (steps & 1) {
      compute(0);
      __syncthreads();     // the next block's tables and the epilogue reuse LDS
    }
  }

  // epilogue: the wave's 64 (n) x 64 (k) block is parked in LDS as fp32 and leaves as 16-byte
  // pieces of 256-byte row segments
  constexpr int ORS = 64 + 4;
  static_assert((size_t)4 * 64 * ORS * sizeof(float) <= kLbWeightLds, "output staging fits in the operand buffers");
  float* tile = reinterpret_cast<float*>(lb_smem) + wv * 64 * ORS;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int jn = 0; jn < 2; ++jn)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const floatx4 f = {acc[i][jn][4 * g], acc[i][jn][4 * g + 1], acc[i][jn][4 * g + 2], acc[i][jn][4 * g + 3]};
        *reinterpret_cast<floatx4*>(&tile[(jn * 32 + l32) * ORS + i * 32 + 8 * g + 4 * hh]) = f;
      }
  __syncthreads();
  float* pw = part_w + (long)split * n_out * K;
  for (int c = lane; c < 64 * 16; c += 64) {
    const int r = c >> 4, ch = c & 15;
    const int n = n0 + wn + r, k = k0 + wk + ch * 4;
    if (n < n_out && k < K)
      *reinterpret_cast<floatx4*>(pw + (long)n * K + k) = *reinterpret_cast<const floatx4*>(&tile[r * ORS + ch * 4]);
  }
  if (do_bias && hh == 0) {
#pragma unroll
    for (int jn = 0; jn < 2; ++jn) {
      const int n = n0 + wn + jn * 32 + l32;
      if (n < n_out) part_b[(long)split * n_out + n] = accb[jn][0];   // every row of the tile holds the column sums
    }
  }
}

// dW = sum of the partial tiles in chunk order; dbias likewise
struct WeightReduceArgs {
  const float *part_w, *part_b;
  const int32_t* total;
  int m_cap, splits;
  long nk;
  int n_out;
  float *dW, *dbias;
};
__device__ __forceinline__ void weight_reduce_block(const WeightReduceArgs& a, unsigned block, unsigned blocks) {
  const int M = a.total != nullptr ? min(a.total[0], a.m_cap) : a.m_cap;
  const int live = token_split(M, a.splits).live;
  const long quads = a.nk >> 2, work = quads + (a.dbias != nullptr ? a.n_out : 0);
  for (long i = (long)block * blockDim.x + threadIdx.x; i < work; i += (long)blocks * blockDim.x) {
    if (i < quads) {
      floatx4 v = {0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < live; ++s) v += *reinterpret_cast<const floatx4*>(a.part_w + (long)s * a.nk + 4 * i);
      *reinterpret_cast<floatx4*>(a.dW + 4 * i) = v;
    } else {
      const long n = i - quads;
      float v = 0.f;
      for (int s = 0; s < live; ++s) v += a.part_b[(long)s * a.n_out + n];
      a.dbias[n] = v;
    }
  }
}
__global__ void __launch_bounds__(256) linear_bwd_weight_reduce_kernel(const WeightReduceArgs a) {
  weight_reduce_block(a, blockIdx.x, gridDim.x);
}
__global__ void __launch_bounds__(256) linear_bwd_weight_reduce_group_kernel(const Members<WeightReduceArgs> m) {
  const MemberBlock mb = member_of(m, blockIdx.x);
  weight_reduce_block(m.a[mb.s], mb.block, mb.blocks);
}

__global__ void __launch_bounds__(256)
linear_bwd_weight_f32_kernel(const float* __restrict__ dout, const int32_t* __restrict__ dout_idx, long ldd,
                             const float* __restrict__ x, const int32_t* __restrict__ x_idx,
                             const float* __restrict__ gate_scores, const int32_t* __restrict__ total, int m_cap, int K,
                             int n_out, float* __restrict__ dW, float* __restrict__ dbias) {
  const int M = total != nullptr ? min(total[0], m_cap) : m_cap;
  const long nk = (long)n_out * K, work = nk + (dbias != nullptr ? n_out : 0);
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < work; i += (long)gridDim.x * blockDim.x) {
    const bool is_w = i < nk;
    const int n = is_w ? (int)(i / K) : (int)(i - nk), k = is_w ? (int)(i - (long)n * K) : 0;
    float a = 0.f;
    for (int m = 0; m < M; ++m) {
      const float g = dout[(dout_idx != nullptr ? (long)dout_idx[m] : (long)m) * ldd + n];
      if (is_w) {
        const long xr = x_idx != nullptr ? (long)x_idx[m] : (long)m;
        const float sc = gate_scores != nullptr ? sigmoidf_dev(gate_scores[xr]) : 1.f;
        a = fmaf(g, sc * x[xr * K + k], a);
      } else {
        a += g;
      }
    }
    if (is_w) dW[i] = a; else dbias[n] = a;
  }
}

static int reserve_lds(const char* fn, const void* kernel, size_t bytes) {
  const hipError_t attr = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  return attr == hipSuccess ? SPA_OK : fail(SPA_ERR_HIP, "%s: cannot reserve %zu bytes of LDS", fn, bytes);
}
// A noted or called weight side: the kernel's arguments but for the shape, the sum of its chunks, where the result goes.
struct WeightCall {
  WeightArgs a;
  WeightReduceArgs r;            // r.part_w, r.part_b: the workspace
  unsigned set(WeightShape s) {  // its workgroups
    a.splits = r.splits = s.splits;
    a.fold = s.fold;
    a.n_tiles = (a.n_out + s.edge - 1) / s.edge;
    a.k_tiles = (a.K + s.edge - 1) / s.edge;
    // one chunk: the tiles are the result; more: partial tiles that the second kernel adds
    r.part_b = r.part_w + (size_t)s.splits * a.n_out * a.K;
    a.part_w = s.splits == 1 ? r.dW : const_cast<float*>(r.part_w);
    a.part_b = s.splits == 1 ? r.dbias : const_cast<float*>(r.part_b);
    return (unsigned)(((long)s.splits * a.n_tiles * a.k_tiles + 7) / 8 * 8);
  }
  unsigned reduce_blocks() const { return (unsigned)std::min<long>((r.nk / 4 + a.n_out + 255) / 256, 4096); }
};

static int launch_weight_big(const char* fn, const WeightPair& p, unsigned blocks, hipStream_t st) {
  if (int rc = reserve_lds(fn, (const void*)weight_gemm_big_kernel, kLbBigLds)) return rc;
  hipLaunchKernelGGL(weight_gemm_big_kernel, dim3(blocks), dim3(512), kLbBigLds, st, p);
  return check_launch(fn);
}
static int launch_weight(const char* fn, WeightCall& c, WeightShape shape, hipStream_t st) {
  const unsigned grid = c.set(shape);
  if (shape.edge == 256) return launch_weight_big(fn, {{c.a, c.a}, grid}, grid, st);
  const bool gi = c.a.dout_idx != nullptr, xi = c.a.x_idx != nullptr;
  const size_t named = (size_t)(gi + xi) * (((c.a.m_cap + shape.splits - 1) / shape.splits + kLbK - 1) / kLbK * kLbK) * sizeof(int);
  if (shape.fold && grid <= 256 && kLbRingLds + named <= kLdsBytes) {
    const auto ring = gi ? (xi ? weight_gemm_ring_kernel<true, true> : weight_gemm_ring_kernel<true, false>)
                         : (xi ? weight_gemm_ring_kernel<false, true> : weight_gemm_ring_kernel<false, false>);
    if (int rc = reserve_lds(fn, (const void*)ring, kLdsBytes)) return rc;      // (one value whatever the call, other threads launch too)
    hipLaunchKernelGGL(ring, dim3(grid), dim3(512), kLbRingLds + named, st, c.a);
    return check_launch(fn);
  }
  const auto kernel = gi ? (xi ? weight_gemm_kernel<true, true> : weight_gemm_kernel<true, false>)
                         : (xi ? weight_gemm_kernel<false, true> : weight_gemm_kernel<false, false>);
  if (int rc = reserve_lds(fn, (const void*)kernel, kLbGemmLds)) return rc;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(kLbThreads), kLbGemmLds, st, c.a);
  return check_launch(fn);
}

// Options gemm_tm and gemm_splits (tuning aids): 2 | 8 forces 128 x 128 | 256 x 256 tiles, 1 to 16 the chunks.
static WeightShape weight_shape(int M_cap, int K, int N_out) {
  return weight_shape(M_cap, K, N_out, options().gemm_tm, options().gemm_splits);
}
static int weight_max_splits(int M_cap, int K, int N_out) {      // (whatever the tiles; rows with a gate scale take the small ones)
  const int forced = options().gemm_splits;
  return std::max({weight_splits(M_cap, K, N_out, forced), weight_most_splits(M_cap, K, N_out, forced), weight_shape(M_cap, K, N_out).splits});
}

// Two weight sides of a group in one launch of 256 x 256 tiles: those of a block past its line, and others that are as large
// and fit the chip at a time.
static bool weights_together(const WeightCall& a, const WeightCall& b) {
  const int cfg = options().gemm_tm;
  if (cfg == 2 || cfg == 8) return cfg == 8;
  long blocks = 0;
  double work = 0;
  for (const WeightCall* c : {&a, &b}) {
    const WeightShape shape = weight_shape(c->a.m_cap, c->a.K, c->a.n_out);
    if (shape.fold) return false;
    blocks += shape.splits * gemm_tiles<long>(c->a.n_out, c->a.K, 256);
    work += weight_work(c->a.m_cap, c->a.K, c->a.n_out);
  }
  return work > kPairWork && blocks <= 256;
}

static thread_local struct {
  int n_rows, n_weight;
  bool big;
  GemmArgs rows;
  WeightCall w[2];
} g_noted;
void group_forget_linear() { g_noted.n_rows = g_noted.n_weight = 0; }
int group_note_rows(const char* fn, const GemmArgs& args, bool big) {
  SPA_REQUIRE(g_noted.n_rows == 0, SPA_ERR_UNSUPPORTED, "%s: one input side in a group", fn);
  g_noted.rows = args;
  g_noted.big = big;
  g_noted.n_rows = 1;
  return SPA_OK;
}
int group_flush_linear(hipStream_t st) {
  auto& n = g_noted;
  const char* fn = "spa_group_end";
  const auto shape = [&](const WeightCall& c) { return weight_shape(c.a.m_cap, c.a.K, c.a.n_out); };
  if (n.n_rows == 1 && n.n_weight > 0 && !n.big) {
    LinearGroup g;
    g.rows = n.rows;
    const long tiles = (long)((n.rows.m_cap + 127) / 128) * ((n.rows.ncols + 127) / 128);
    g.end[0] = (unsigned)((tiles + 7) / 8 * 8);
    unsigned blocks = g.end[0];
    // long chunks first: what does not fit at a time comes last, and short
    if (n.n_weight == 2 && shape(n.w[0]).splits > shape(n.w[1]).splits) std::swap(n.w[0], n.w[1]);
    for (int i = 0; i < n.n_weight; ++i) {
      const WeightShape own = shape(n.w[i]);
      blocks += n.w[i].set({kLbT, own.splits, own.fold});
      if (i == 0) g.end[1] = blocks;
      g.w[i] = n.w[i].a;
    }
    if (n.n_weight == 1) g.w[1] = g.w[0];
    if (int rc = reserve_lds(fn, (const void*)linear_bwd_group_kernel, kLbGemmLds)) return rc;
    hipLaunchKernelGGL(linear_bwd_group_kernel, dim3(blocks), dim3(kLbThreads), kLbGemmLds, st, g);
  } else {
    if (n.n_rows == 1)
      if (int rc = launch_gemm_rows(fn, n.rows, true, st)) return rc;
    if (n.n_weight == 2 && weights_together(n.w[0], n.w[1])) {
      WeightPair p;
      unsigned blocks = 0;
      for (int i = 0; i < 2; ++i) {
        blocks += n.w[i].set({256, shape(n.w[i]).splits});
        if (i == 0) p.end = blocks;
        p.w[i] = n.w[i].a;
      }
      if (int rc = launch_weight_big(fn, p, blocks, st)) return rc;
    } else {
      for (int i = 0; i < n.n_weight; ++i)
        if (int rc = launch_weight(fn, n.w[i], shape(n.w[i]), st)) return rc;
    }
  }
  Noted<WeightReduceArgs> reduce;
  for (int i = 0; i < n.n_weight; ++i)
    if (n.w[i].r.splits > 1)
      if (int rc = reduce.add(fn, n.w[i].r, n.w[i].reduce_blocks())) return rc;
  if (reduce.n > 0) {
    Members<WeightReduceArgs> m;
    const unsigned blocks = reduce.members(m);
    hipLaunchKernelGGL(linear_bwd_weight_reduce_group_kernel, dim3(blocks), dim3(256), 0, st, m);
  }
  return check_launch(fn);
}

}  // namespace spa

using namespace spa;

extern "C" int spa_linear_packed_bwd_input(const void* dout, const int32_t* dout_idx, int64_t dout_row_stride,
                                           const int32_t* total, const void* W, int M_cap, int K, int N_out, int dtype,
                                           const int32_t* dx_idx, const int32_t* inv_pos, int64_t rows, void* dx,
                                           int64_t dx_row_stride, void* stream) {
  const char* fn = "spa_linear_packed_bwd_input";
  SPA_REQUIRE(dout && W && dx, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(M_cap >= 1 && K >= 1 && N_out >= 1, SPA_ERR_INVALID_ARG, "%s: M_cap, K, N_out must be >= 1", fn);
  SPA_REQUIRE(dtype == SPA_F32 || dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: unknown dtype %d", fn, dtype);
  SPA_REQUIRE(dout_row_stride >= N_out && dx_row_stride >= K, SPA_ERR_INVALID_ARG,
              "%s: dout_row_stride < N_out or dx_row_stride < K", fn);
  SPA_REQUIRE(inv_pos == nullptr || (dx_idx != nullptr && rows >= 0), SPA_ERR_INVALID_ARG,
              "%s: inv_pos (zero fill of the rows no packed row maps to) needs dx_idx and rows >= 0", fn);
  hipStream_t st = as_stream(stream);
  SPA_REQUIRE(!(group_open() && dtype == SPA_F32), SPA_ERR_UNSUPPORTED, "%s: fp32 calls cannot be part of a group", fn);
  if (dtype == SPA_F32) {
    long work = (long)M_cap * K;
    if (inv_pos != nullptr && rows * K > work) work = rows * K;
    long wgs = (work + 255) / 256;
    if (wgs > 8192) wgs = 8192;
    hipLaunchKernelGGL(linear_bwd_input_f32_kernel, dim3((unsigned)wgs), dim3(256), 0, st, (const float*)dout, dout_idx,
                       (long)dout_row_stride, total, (const float*)W, M_cap, N_out, K, (float*)dx, (long)dx_row_stride,
                       dx_idx, inv_pos, (long)rows);
    return check_launch(fn);
  }
  SPA_REQUIRE(K % 8 == 0 && N_out % 8 == 0 && dout_row_stride % 8 == 0 && dx_row_stride % 8 == 0, SPA_ERR_UNSUPPORTED,
              "%s: K, N_out and the row strides must be multiples of 8 for bf16", fn);
  SPA_REQUIRE(aligned16(dout) && aligned16(W) && aligned16(dx), SPA_ERR_INVALID_ARG,
              "%s: dout / W / dx not 16-byte aligned", fn);
  GemmArgs args = {};
  args.a = (const __bf16*)dout;
  args.a_idx = dout_idx;
  args.lda = dout_row_stride;
  args.total = total;
  args.m_cap = M_cap;
  args.kc = N_out;
  args.ncols = K;
  args.w = (const __bf16*)W;
  args.out = (__bf16*)dx;
  args.ldo = dx_row_stride;
  args.o_idx = dx_idx;
  args.inv_pos = inv_pos;
  args.zrows = rows;
  return launch_gemm_rows(fn, args, true, st);
}

extern "C" size_t spa_linear_bwd_weight_workspace_bytes(int M_cap, int K, int N_out, int dtype) {
  if (dtype != SPA_BF16 || M_cap < 1 || K < 1 || N_out < 1) return 0;
  const size_t per_split = ((size_t)N_out * K + N_out) * sizeof(float);
  return ((size_t)weight_max_splits(M_cap, K, N_out) * per_split + 255) & ~(size_t)255;
}

extern "C" int spa_linear_packed_bwd_weight(const void* dout, const int32_t* dout_idx, int64_t dout_row_stride,
                                            const void* x, const int32_t* x_idx, const float* gate_scores,
                                            const int32_t* total, int M_cap, int K, int N_out, int dtype, float* dW,
                                            float* dbias, void* workspace, size_t workspace_bytes, void* stream) {
  const char* fn = "spa_linear_packed_bwd_weight";
  SPA_REQUIRE(dout && x && dW, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(M_cap >= 1 && K >= 1 && N_out >= 1, SPA_ERR_INVALID_ARG, "%s: M_cap, K, N_out must be >= 1", fn);
  SPA_REQUIRE(dtype == SPA_F32 || dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: unknown dtype %d", fn, dtype);
  SPA_REQUIRE(dout_row_stride >= N_out, SPA_ERR_INVALID_ARG, "%s: dout_row_stride < N_out", fn);
  SPA_REQUIRE(!(gate_scores != nullptr && x_idx == nullptr), SPA_ERR_INVALID_ARG,
              "%s: gate_scores are indexed by token and need x_idx", fn);
  hipStream_t st = as_stream(stream);
  SPA_REQUIRE(!(group_open() && dtype == SPA_F32), SPA_ERR_UNSUPPORTED, "%s: fp32 calls cannot be part of a group", fn);
  if (dtype == SPA_F32) {
    long wgs = ((long)N_out * K + N_out + 255) / 256;
    if (wgs > 8192) wgs = 8192;
    hipLaunchKernelGGL(linear_bwd_weight_f32_kernel, dim3((unsigned)wgs), dim3(256), 0, st, (const float*)dout, dout_idx,
                       (long)dout_row_stride, (const float*)x, x_idx, gate_scores, total, M_cap, K, N_out, dW, dbias);
    return check_launch(fn);
  }
  SPA_REQUIRE(K % 8 == 0 && N_out % 8 == 0 && dout_row_stride % 8 == 0, SPA_ERR_UNSUPPORTED,
              "%s: K, N_out and dout_row_stride must be multiples of 8 for bf16", fn);
  SPA_REQUIRE(aligned16(dout) && aligned16(x) && aligned16(dW), SPA_ERR_INVALID_ARG,
              "%s: dout / x / dW not 16-byte aligned", fn);
  const size_t need = spa_linear_bwd_weight_workspace_bytes(M_cap, K, N_out, dtype);
  SPA_REQUIRE(workspace != nullptr && workspace_bytes >= need, SPA_ERR_WORKSPACE,
              "%s: workspace of %zu bytes needed, %zu given", fn, need, workspace_bytes);
  SPA_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255u) == 0, SPA_ERR_INVALID_ARG,
              "%s: workspace not 256-byte aligned", fn);
  const WeightShape shape = gate_scores != nullptr ? WeightShape{kLbT, weight_splits(M_cap, K, N_out, options().gemm_splits)} : weight_shape(M_cap, K, N_out);
  SPA_REQUIRE(shape.splits * shape.tiles(N_out, K) + 8 < 2147483647L / 2, SPA_ERR_INVALID_ARG, "%s: too many tiles", fn);
  SPA_REQUIRE(!(group_open() && gate_scores != nullptr), SPA_ERR_UNSUPPORTED, "%s: gated rows cannot be part of a group", fn);
  WeightCall c = {};
  c.a.dout = (const __bf16*)dout;
  c.a.dout_idx = dout_idx;
  c.a.ldd = dout_row_stride;
  c.a.x = (const __bf16*)x;
  c.a.x_idx = x_idx;
  c.a.total = total;
  c.a.m_cap = M_cap;
  c.a.K = K;
  c.a.n_out = N_out;
  c.r = {static_cast<const float*>(workspace), nullptr, total, M_cap, 0, (long)N_out * K, N_out, dW, dbias};
  if (group_open()) {
    SPA_REQUIRE(g_noted.n_weight < 2, SPA_ERR_UNSUPPORTED, "%s: two weight sides in a group", fn);
    g_noted.w[g_noted.n_weight++] = c;
    return SPA_OK;
  }
  if (gate_scores != nullptr) {
    const unsigned grid = c.set(shape);
    if (int rc = reserve_lds(fn, (const void*)linear_bwd_weight_bf16_kernel, kLbWeightLds)) return rc;
    hipLaunchKernelGGL(linear_bwd_weight_bf16_kernel, dim3(grid), dim3(kLbThreads), kLbWeightLds, st, c.a.dout, dout_idx, c.a.ldd,
                       c.a.x, x_idx, gate_scores, total, M_cap, K, N_out, shape.splits, c.a.n_tiles, c.a.k_tiles,
                       const_cast<float*>(c.r.part_w), const_cast<float*>(c.r.part_b));
  } else {
    if (int rc = launch_weight(fn, c, shape, st)) return rc;
    if (shape.splits == 1) return SPA_OK;
  }
  const int rc = check_launch(fn);
  if (rc != SPA_OK) return rc;
  hipLaunchKernelGGL(linear_bwd_weight_reduce_kernel, dim3(c.reduce_blocks()), dim3(256), 0, st, c.r);
  return check_launch(fn);
}

