// Linear projection of packed tokens (the 3 L C^2 and N C^2 terms of the SPA complexity
// formula, Section 3.2): out[j,:] = (s_j * x[row(j),:]) W^T + bias, where row(j) is either j
// or gather_idx[j] (the token gather of the packing step folded into the A-operand load) and
// s_j is 1 or sigmoid(score) of the token (the gated representation r_g = Sigmoid(s) . r).
// The row scale s_j is applied to the fp32 accumulator in the epilogue: (s a) W^T = s (a W^T),
// one rounding fewer than multiplying a materialised bf16 r_g.
//
// bf16 path: MFMA GEMM on the pipelined loop of gemm_async.h, 64 deep steps, tiles of 128 x 128 (four waves
// of 64 x 64, two workgroups per unit; eight of 64 x 32 where a unit has one tile, or about one), 192 x 192, 256 x 192 or 256 x 256
// (eight waves); the same kernels multiply by W as it lies for the input side of the backward (linear_bwd.hip).  With 128 x 128 tiles every flop
// needs 1/64 byte from L2; the large tiles need two thirds and half of that and win wherever they still fill the chip
// (gemm_shape.h; what bounds them: gemm_rows.h).  Measured, called again and again: 12544 rows of 768 -> 2304 47 to 49 us =
// 905 to 940 TFLOP/s (operands staged through registers: 68 us); 6272 rows of 384 -> 384: 7 us (8.7); 98 rows: 5.8 us (8.1),
// its steps bound by latency.  The output tile leaves through LDS as whole rows.
// fp32 path (tiny workload): one thread per output element.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "gemm_rows.h"
#include "group.h"
#include "spa_common.h"

namespace spa {

template <bool kGather, bool kScale>
__global__ void __launch_bounds__(256)
linear_f32_kernel(const float* __restrict__ x, const int32_t* __restrict__ gather_idx,
                  const float* __restrict__ gate_scores, const int32_t* __restrict__ total,
                  const float* __restrict__ W, const float* __restrict__ bias, int m_cap, int K, int n_out,
                  float* out, long out_stride, const int32_t* __restrict__ scatter_idx, const float* residual,
                  const int32_t* __restrict__ inv_pos, long rows) {
  if (inv_pos != nullptr)          // the rows no packed row maps to keep the residual
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < rows * n_out; i += (long)gridDim.x * blockDim.x) {
      const long r = i / n_out, at = r * out_stride + (i - r * n_out);
      if (inv_pos[r] < 0) out[at] = residual[at];
    }
  const int M = total != nullptr ? min(total[0], m_cap) : m_cap;
  const long work = (long)M * n_out;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < work; i += (long)gridDim.x * blockDim.x) {
    const int m = (int)(i / n_out), n = (int)(i - (long)m * n_out);
    const long src = kGather ? (long)gather_idx[m] : (long)m;
    const float sc = kScale ? sigmoidf_dev(gate_scores[src]) : 1.f;
    const float* xr = x + src * K;
    const float* wr = W + (long)n * K;
    float a = 0.f;
    for (int kq = 0; kq < K; ++kq) a = fmaf(sc * xr[kq], wr[kq], a);
    const long off = (long)(scatter_idx != nullptr ? scatter_idx[m] : m) * out_stride + n;
    out[off] = a + (bias != nullptr ? bias[n] : 0.f) + (residual != nullptr ? residual[off] : 0.f);
  }
}

template <bool kScale, bool kDeep>
static int launch_gemm_rows_tile(const char* fn, GemmArgs args, bool big, hipStream_t st) {
  args.rule = large_rule(args.ncols, args.kc, args.residual != nullptr);
  const bool ring = !big && ring_tiles(args.m_cap, args.total != nullptr, args.ncols);
  const bool eight = !big && two_rings(args.m_cap, args.total != nullptr, args.ncols, args.kc);
  const size_t smem = big ? kGemmBigLds : ring && !eight ? kGemmRingLds : kGemmSmallLds;
  const long tiles = gemm_tiles<long>(args.m_cap, args.ncols, big ? 192 : 128);     // (no less than with 256)
  SPA_REQUIRE(tiles + 8 < 2147483647L / 2, SPA_ERR_INVALID_ARG, "%s: too many tiles", fn);
  const long tiles8 = (tiles + 7) / 8 * 8;
  const int cfg = options().gemm_tm;
  const auto large = cfg == 6    ? gemm_rows_big_kernel<kScale, kDeep, Large::k192>
                     : cfg == 8  ? gemm_rows_big_kernel<kScale, kDeep, Large::k256>
                     : cfg == 10 ? gemm_rows_big_kernel<kScale, kDeep, Large::k256x192>
                                 : gemm_rows_big_kernel<kScale, kDeep, Large::kByRows>;
  const auto kernel = big     ? large
                      : eight ? gemm_rows_eight_kernel<kScale, kDeep>
                      : ring  ? gemm_rows_ring_kernel<kScale, kDeep>
                              : gemm_rows_small_kernel<kScale, kDeep>;
  const hipError_t attr = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  SPA_REQUIRE(attr == hipSuccess, SPA_ERR_HIP, "%s: cannot reserve %zu bytes of LDS", fn, smem);
  hipLaunchKernelGGL(kernel, dim3((unsigned)(big ? std::min(tiles8, 256L) : tiles8)), dim3(big || ring ? 512 : 256), smem, st, args);
  return check_launch(fn);
}

// Option gemm_tm (tuning aid) forces a shape: 2 | 6 | 8 | 10 for 128 x 128 | 192 x 192 | 256 x 256 | 256 x 192, 14 for the
// large ones by the live rows.
int launch_gemm_rows(const char* fn, const GemmArgs& args, bool deep, hipStream_t st) {
  const int cfg = options().gemm_tm;
  const bool big = cfg != 0 ? cfg >= 6 : large_tiles(args.m_cap, args.total != nullptr, args.ncols, args.kc);
  if (group_open()) return group_note_rows(fn, args, big);
  if (deep) return launch_gemm_rows_tile<false, true>(fn, args, big, st);
  if (args.scores != nullptr) return launch_gemm_rows_tile<true, false>(fn, args, big, st);
  return launch_gemm_rows_tile<false, false>(fn, args, big, st);
}

}  // namespace spa

using namespace spa;

static int linear_common(const char* fn, const void* x, const int32_t* gather_idx, const float* gate_scores,
                         const int32_t* total, const void* W, const void* bias, int M_cap, int K, int N_out,
                         int dtype, void* out, int64_t out_row_stride, const int32_t* scatter_idx,
                         const void* residual, const int32_t* inv_pos, int64_t rows, void* stream) {
  SPA_REFUSE_IN_GROUP(fn);
  SPA_REQUIRE(x && W && out, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(M_cap >= 1 && K >= 1 && N_out >= 1, SPA_ERR_INVALID_ARG, "%s: M_cap, K, N_out must be >= 1", fn);
  SPA_REQUIRE(dtype == SPA_F32 || dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: unknown dtype %d", fn, dtype);
  SPA_REQUIRE(!(gate_scores != nullptr && gather_idx == nullptr), SPA_ERR_INVALID_ARG,
              "%s: gate_scores are indexed by token and need gather_idx", fn);
  SPA_REQUIRE(out_row_stride >= N_out, SPA_ERR_INVALID_ARG, "%s: out_row_stride < N_out", fn);
  hipStream_t st = as_stream(stream);
  const bool g = gather_idx != nullptr, sc = gate_scores != nullptr;
  if (dtype == SPA_F32) {
    long wgs = (std::max((long)M_cap, inv_pos != nullptr ? (long)rows : 0L) * N_out + 255) / 256;
    if (wgs > 8192) wgs = 8192;
#define SPA_LIN_F32(G_, S_)                                                                                   \
  hipLaunchKernelGGL((linear_f32_kernel<G_, S_>), dim3((unsigned)wgs), dim3(256), 0, st, (const float*)x,    \
                     gather_idx, gate_scores, total, (const float*)W, (const float*)bias, M_cap, K, N_out,   \
                     (float*)out, (long)out_row_stride, scatter_idx, (const float*)residual, inv_pos, (long)rows)
    if (g && sc) SPA_LIN_F32(true, true); else if (g) SPA_LIN_F32(true, false); else SPA_LIN_F32(false, false);
#undef SPA_LIN_F32
    return check_launch(fn);
  }
  SPA_REQUIRE(K % 8 == 0, SPA_ERR_UNSUPPORTED, "%s: K = %d must be a multiple of 8 for bf16", fn, K);
  SPA_REQUIRE(N_out % 8 == 0 && out_row_stride % 8 == 0, SPA_ERR_INVALID_ARG,
              "%s: N_out and out_row_stride must be multiples of 8 for bf16", fn);
  SPA_REQUIRE(aligned16(x) && aligned16(W) && aligned16(out), SPA_ERR_INVALID_ARG, "%s: x / W / out not 16-byte aligned", fn);
  GemmArgs args = {};
  args.a = (const __bf16*)x;
  args.a_idx = gather_idx;
  args.lda = K;
  args.scores = gate_scores;
  args.total = total;
  args.m_cap = M_cap;
  args.kc = K;
  args.ncols = N_out;
  args.w = (const __bf16*)W;
  args.bias = (const __bf16*)bias;
  args.out = (__bf16*)out;
  args.ldo = out_row_stride;
  args.o_idx = scatter_idx;
  args.residual = (const __bf16*)residual;
  args.inv_pos = inv_pos;
  args.zrows = rows;
  return launch_gemm_rows(fn, args, false, st);
}

extern "C" int spa_linear_packed(const void* x, const int32_t* gather_idx, const float* gate_scores,
                                 const int32_t* total, const void* W, const void* bias, int M_cap, int K,
                                 int N_out, int dtype, void* out, int64_t out_row_stride, void* stream) {
  return linear_common("spa_linear_packed", x, gather_idx, gate_scores, total, W, bias, M_cap, K, N_out, dtype, out,
                       out_row_stride, nullptr, nullptr, nullptr, 0, stream);
}

extern "C" int spa_linear_packed_scatter(const void* x, const int32_t* total, const void* W, const void* bias,
                                         int M_cap, int K, int N_out, int dtype, const int32_t* scatter_idx,
                                         const void* residual, void* y, int64_t y_row_stride, void* stream) {
  const char* fn = "spa_linear_packed_scatter";
  SPA_REQUIRE(scatter_idx != nullptr, SPA_ERR_INVALID_ARG, "%s: scatter_idx is null", fn);
  SPA_REQUIRE(aligned16(residual), SPA_ERR_INVALID_ARG, "%s: residual not 16-byte aligned", fn);
  return linear_common(fn, x, nullptr, nullptr, total, W, bias, M_cap, K, N_out, dtype, y, y_row_stride, scatter_idx,
                       residual, nullptr, 0, stream);
}

extern "C" int spa_linear_packed_unpack(const void* x, const int32_t* total, const void* W, const void* bias, int M_cap,
                                        int K, int N_out, int dtype, const int32_t* gather_idx, const int32_t* inv_pos,
                                        int64_t rows, const void* residual, void* y, void* stream) {
  const char* fn = "spa_linear_packed_unpack";
  SPA_REQUIRE(gather_idx && inv_pos && residual, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(rows >= 1 && rows < 2147483647L, SPA_ERR_INVALID_ARG, "%s: rows must be in [1, 2^31)", fn);
  SPA_REQUIRE(aligned16(residual), SPA_ERR_INVALID_ARG, "%s: residual not 16-byte aligned", fn);
  return linear_common(fn, x, nullptr, nullptr, total, W, bias, M_cap, K, N_out, dtype, y, N_out, gather_idx, residual,
                       inv_pos, rows, stream);
}
