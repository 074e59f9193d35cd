// Backward of the packed, per-image attention: for every (image, head) segment
//   P = exp(S - lse), dV = P^T dO, dP = dO V^T, D_i = sum_d dO_id O_id,
//   dS = P * (dP - D), dQ = dS K * scale, dK = dS^T Q * scale.
// No atomics anywhere; results are run-to-run bit-stable.
// Segments of up to 256 tokens (bf16): one kernel, a workgroup per (image, head); see
// attn_bwd_short_bf16_kernel.
// Longer segments (bf16): two roles in one launch, after a small kernel that writes D_i (or the forward pass has):
//   dq role   : a wave owns 32 queries and walks the segment's keys.  Like the forward it
//               works on transposed tiles (S^T = K Q^T, dP^T = V dO^T) so lse_i and D_i are
//               one scalar per lane and dS^T is already the B operand of dQ^T += K^T dS^T.
//   dkdv role : a wave owns 32 keys and walks the segment's queries with S = Q K^T and
//               dP = dO V^T un-transposed (lane = key), so P and dS are the B operands of
//               dV^T += dO^T P and dK^T += Q^T dS.
//   S and dP are recomputed in both roles (7 GEMM shapes instead of 5) in exchange for
//   determinism.
// fp32: a thread per row (query side, then key side), the other side streaming through LDS.
// Every form can read the upstream gradient and write dq, dk, dv at token positions (TokenIO).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "attn_tiles.h"
#include "group.h"
#include "spa_common.h"

namespace spa {

constexpr float kLog2e = 1.4426950408889634f;

struct Seg {
  long row0;
  int n;
};
__device__ __forceinline__ Seg seg_of(int b, const int32_t* cu) {
  Seg s;
  const int a = cu[b];
  s.row0 = a;
  s.n = cu[b + 1] - a;
  return s;
}


// Token-position I/O folded into the kernel (gather_idx == nullptr: packed I/O): the upstream
// gradient row of packed token j is dy[gather_idx[j]], the gradients of packed token j go to
// row gather_idx[j] of dq / dk / dv, and the rows of unselected tokens (inv_pos < 0) are zeroed,
// every workgroup of the launch clearing an even share (short segments: its head's columns).
struct TokenIO {
  const int32_t* gather_idx;
  const int32_t* inv_pos;
  long rows;               // B * N
};

// The wave's transposed accumulator tile (rows = head dim, a lane = one token) as bf16 rows: the two halves
// of the wave exchange quads so that a lane holds 8 consecutive columns of its token, 16-byte stores.
template <int DH>
__device__ __forceinline__ void store_rows(const floatx16 (&acc)[DH / 32], float scale, __bf16* row, bool ok, int hh) {
#pragma unroll
  for (int d = 0; d < DH / 32; ++d)
#pragma unroll
    for (int g = 0; g < 4; g += 2) {
      uint32_t w[2][2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const floatx4 f = {acc[d][4 * (g + u)] * scale, acc[d][4 * (g + u) + 1] * scale, acc[d][4 * (g + u) + 2] * scale,
                           acc[d][4 * (g + u) + 3] * scale};
        const uintx2 p = __builtin_bit_cast(uintx2, __builtin_convertvector(f, bf16x4));
        w[u][0] = p[0];
        w[u][1] = p[1];
      }
      // lanes 32.. of the first quad <-> lanes ..31 of the second
      const auto x0 = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
      const auto x1 = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
      const uintx4 v = {x0[0], x1[0], x0[1], x1[1]};
      if (ok) *reinterpret_cast<uintx4*>(row + d * 32 + 8 * g + 8 * hh) = v;
    }
}

// Operands and results of the bf16 kernels.
struct BwdArgs {
  const __bf16 *q, *k, *v;
  long qs, ks, vs;
  const float* v_scores;         // GATED: score of every token
  const __bf16 *out, *dout;      // out: packed rows
  const float* lse;
  long lse_stride;
  const int32_t* cu;
  int H, B;
  float scale;
  __bf16 *dq, *dk, *dv;
  long dqs, dks, dvs;
  TokenIO tok;
  float* dvec;                   // long segments: D_i for every (head, packed row)
  int nblk;                      // long segments: blocks of kBwdRows rows of the longest possible one
};

// -------------------------------------------------------------------------- long segments (bf16)
constexpr int kBwdBT = 64, kBwdThreads = 256, kBwdRows = 128;     // streamed tile, 4 waves x 32 rows

// Rows of the long kernel's operands: q, k, v, out packed, dO and the gradients
//   kPacked: packed as well;  kTokens: at token positions;  kGated: q, k, v at token positions too, v gated.
enum BwdRowsMode { kPacked, kTokens, kGated };

template <int DH>
struct BwdLongLds {
  static constexpr int RS = DH + 8;
  __attribute__((aligned(16))) __bf16 A[2][kBwdBT * RS];         // K (dq) | Q (dkdv)
  __attribute__((aligned(16))) __bf16 Bm[2][kBwdBT * RS];        // V (dq) | dO (dkdv)
  __attribute__((aligned(16))) float lse2s[2][kBwdBT];           // of the streamed queries (dkdv)
  __attribute__((aligned(16))) float negD[2][kBwdBT];
};

// Scores and dP of the wave's 32 tokens of the streamed tile against its 32 rows: two chains of DH / 16
// MFMAs; dp starts from c (-D, so that dS = P dP needs no subtraction), s
// from what it holds.
template <int DH>
__device__ __forceinline__ void bwd_scores(const __bf16* at, const __bf16* bt, int sb, const bf16x8 (&af)[DH / 16],
                                           const bf16x8 (&bf)[DH / 16], const floatx16& c, floatx16& s, floatx16& dp, int l32,
                                           int hh) {
  constexpr int RS = DH + 8;
  dp = c;
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk) {
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(&at[(sb * 32 + l32) * RS + kk * 16 + hh * 8]);
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, af[kk], s, 0, 0, 0);
    const bf16x8 y = *reinterpret_cast<const bf16x8*>(&bt[(sb * 32 + l32) * RS + kk * 16 + hh * 8]);
    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y, bf[kk], dp, 0, 0, 0);
  }
}

// (LOOP: the role is called in a loop over blocks.)
// dq role: 32 queries per wave against the keys of the segment.  S^T = K Q^T, dP^T = V dO^T: a lane holds 16
// keys of one query, lse and D are one scalar per lane, dS^T is the B operand of dQ^T += K^T dS^T.
template <int DH, int MODE, bool LOOP>
__device__ __forceinline__ void bwd_dq_role(BwdLongLds<DH>& lds, const BwdArgs& p, const Segment seg, int h, int q0) {
  constexpr int RS = DH + 8, KK = DH / 16, DB = DH / 32, BT = kBwdBT;
  constexpr bool GATED = MODE == kGated;
  using Stage = PairStage<DH, kBwdThreads, BT, GATED, GATED>;
  const int tid = LOOP ? fresh_thread_id() : threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
  const int qi = q0 + wv * 32 + l32, n = seg.nk;
  const bool wave_live = q0 + wv * 32 < n, q_ok = qi < n;
  const long C = (long)p.H * DH;
  const float scale_log2 = p.scale * kLog2e;
  const int32_t* gi = MODE != kPacked ? p.tok.gather_idx + seg.row0 : nullptr;
  const long q_row = seg.row0 + (q_ok ? qi : 0);
  const long tok_row = MODE != kPacked ? (long)gi[q_ok ? qi : 0] : q_row;

  Stage st(tid);
  float gate[Stage::CPT] = {};
  st.gi = gi;
  st.last = n - 1;
  st.source(0, p.k + h * DH, p.ks, seg.row0);
  st.source(1, p.v + h * DH, p.vs, seg.row0);
  auto load_tile = [&](int kt) {                     // (then the index of the one after it)
    st.load(kt);
    if (GATED) {
#pragma unroll
      for (int t = 0; t < Stage::CPT; ++t) gate[t] = p.v_scores[st.idx[t]];
    }
    st.index(kt + BT);
  };
  st.index(0);
  load_tile(0);
  bf16x8 qf[KK], dof[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int col = h * DH + kk * 16 + hh * 8;
    qf[kk] = zero_bf16x8();
    dof[kk] = zero_bf16x8();
    if (q_ok) {
      qf[kk] = *reinterpret_cast<const bf16x8*>(p.q + (GATED ? tok_row : q_row) * p.qs + col);
      dof[kk] = *reinterpret_cast<const bf16x8*>(p.dout + tok_row * C + col);
    }
  }
  const float negd = q_ok ? -p.dvec[h * p.lse_stride + q_row] : 0.f;
  const float lse2 = q_ok ? p.lse[h * p.lse_stride + q_row] * kLog2e : INFINITY;   // past the segment: probability 0
  floatx16 acc[DB], negD;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    negD[r] = negd;
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[d][r] = 0.f;
  }
  auto store_tile = [&](int buf, auto clear) {
    if (GATED) st.template store_gated<clear>(lds.A[buf], lds.Bm[buf], gate);
    else st.template store<clear>(lds.A[buf], lds.Bm[buf]);
  };
  store_tile(0, std::true_type{});
  __syncthreads();
  const int nt = (n + BT - 1) / BT;
  walk_tiles(nt, [&](int t, auto at) {
    constexpr bool last = decltype(at)::value == kTileLast;
    const int buf = t & 1, kt = t * BT;
    if (!last) load_tile(kt + BT);
    if (wave_live) {
      floatx16 s[2], dp[2];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[sb][r] = 0.f;
        bwd_scores<DH>(lds.A[buf], lds.Bm[buf], sb, qf, dof, negD, s[sb], dp[sb], l32, hh);
      }
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        if (last) {
          const int left = n - kt - sb * 32;         // valid keys of the sub-block
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (acc_row(r, hh) >= left) s[sb][r] = -INFINITY;
        }
#pragma unroll
        for (int mf = 0; mf < 2; ++mf) {
          floatx8 f;
#pragma unroll
          for (int j = 0; j < 8; ++j)
            f[j] = __builtin_amdgcn_exp2f(fmaf(s[sb][8 * mf + j], scale_log2, -lse2)) * dp[sb][8 * mf + j];
          const bf16x8 dsb = float_to_bf16x8(f);
#pragma unroll
          for (int d = 0; d < DB; ++d)
            acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(transposed_frag_rowmajor<RS>(lds.A[buf], d, sb * 32, mf, lane), dsb,
                                                             acc[d], 0, 0, 0);
        }
      }
    }
    if (!last) {
      store_tile(buf ^ 1, std::bool_constant<decltype(at)::value == kTileBeforeLast>{});
      __syncthreads();
    }
  });
  store_rows<DH>(acc, p.scale, p.dq + tok_row * p.dqs + h * DH, q_ok, hh);
}

// dkdv role: 32 keys per wave against the queries.  S = Q K^T, dP = dO V^T: a lane holds 16 queries of one
// key, P and dS are the B operands of dV^T += dO^T P and dK^T += Q^T dS.
template <int DH, int MODE, bool LOOP>
__device__ __forceinline__ void bwd_dkdv_role(BwdLongLds<DH>& lds, const BwdArgs& p, const Segment seg, int h, int k0) {
  constexpr int RS = DH + 8, KK = DH / 16, DB = DH / 32, BT = kBwdBT;
  constexpr bool GATED = MODE == kGated;
  using Stage = PairStage<DH, kBwdThreads, BT, GATED, MODE != kPacked>;
  const int tid = LOOP ? fresh_thread_id() : threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
  const int ki = k0 + wv * 32 + l32, n = seg.nk;
  const bool wave_live = k0 + wv * 32 < n, k_ok = ki < n;
  const long C = (long)p.H * DH;
  const float scale_log2 = p.scale * kLog2e;
  const int32_t* gi = MODE != kPacked ? p.tok.gather_idx + seg.row0 : nullptr;
  const float* lse_h = p.lse + h * p.lse_stride + seg.row0;
  const float* dvec_h = p.dvec + h * p.lse_stride + seg.row0;
  const long k_row = seg.row0 + (k_ok ? ki : 0);
  const long tok_row = MODE != kPacked ? (long)gi[k_ok ? ki : 0] : k_row, src = GATED ? tok_row : k_row;

  Stage st(tid);
  st.gi = gi;
  st.last = n - 1;
  st.source(0, p.q + h * DH, p.qs, seg.row0);
  st.source(1, p.dout + h * DH, C, seg.row0);
  float lse_t = 0.f, d_t = 0.f;                      // of streamed query `lane` of the tile
  auto load_tile = [&](int qt) {                     // (then the index of the one after it)
    st.load(qt);
    st.index(qt + BT);
    const int q = min(qt + lane, n - 1);
    lse_t = lse_h[q];
    d_t = dvec_h[q];
  };
  auto store_all = [&](int buf, int qt, auto clear) {
    st.template store<clear>(lds.A[buf], lds.Bm[buf]);
    if (tid < BT) {
      lds.lse2s[buf][tid] = qt + tid < n ? lse_t * kLog2e : INFINITY;    // past the segment: probability 0
      lds.negD[buf][tid] = -d_t;
    }
  };
  st.index(0);
  load_tile(0);
  bf16x8 kf[KK], vf[KK];
  const float gate = GATED && k_ok ? sigmoidf_dev(p.v_scores[src]) : 1.f;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int col = h * DH + kk * 16 + hh * 8;
    kf[kk] = zero_bf16x8();
    vf[kk] = zero_bf16x8();
    if (k_ok) {
      kf[kk] = *reinterpret_cast<const bf16x8*>(p.k + src * p.ks + col);
      vf[kk] = *reinterpret_cast<const bf16x8*>(p.v + src * p.vs + col);
      if (GATED) vf[kk] = scale_row(vf[kk], gate);
    }
  }
  floatx16 dka[DB], dva[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dka[d][r] = 0.f; dva[d][r] = 0.f; }
  store_all(0, 0, std::true_type{});
  __syncthreads();
  const int nt = (n + BT - 1) / BT;
  walk_tiles(nt, [&](int t, auto at) {
    constexpr bool last = decltype(at)::value == kTileLast;
    const int buf = t & 1, qt = t * BT;
    if (!last) load_tile(qt + BT);
    if (wave_live) {
      const __bf16 *qb = lds.A[buf], *gb = lds.Bm[buf];
      floatx16 s[2], dp[2];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        floatx16 c;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const floatx4 d4 = *reinterpret_cast<const floatx4*>(&lds.negD[buf][sb * 32 + 8 * g + 4 * hh]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            c[4 * g + e] = d4[e];
            s[sb][4 * g + e] = 0.f;
          }
        }
        bwd_scores<DH>(qb, gb, sb, kf, vf, c, s[sb], dp[sb], l32, hh);
      }
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int mf = 0; mf < 2; ++mf) {
          floatx8 fp, fd;
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const floatx4 l4 = *reinterpret_cast<const floatx4*>(&lds.lse2s[buf][sb * 32 + 16 * mf + 8 * g + 4 * hh]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int j = 4 * g + e;
              fp[j] = __builtin_amdgcn_exp2f(fmaf(s[sb][8 * mf + j], scale_log2, -l4[e]));
              fd[j] = fp[j] * dp[sb][8 * mf + j];
            }
          }
          const bf16x8 pb = float_to_bf16x8(fp), dsb = float_to_bf16x8(fd);
#pragma unroll
          for (int d = 0; d < DB; ++d) {
            dva[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(transposed_frag_rowmajor<RS>(gb, d, sb * 32, mf, lane), pb, dva[d], 0, 0, 0);
            dka[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(transposed_frag_rowmajor<RS>(qb, d, sb * 32, mf, lane), dsb, dka[d], 0, 0, 0);
          }
        }
    }
    if (!last) {
      store_all(buf ^ 1, qt + BT, std::bool_constant<decltype(at)::value == kTileBeforeLast>{});
      __syncthreads();
    }
  });
  store_rows<DH>(dka, p.scale, p.dk + tok_row * p.dks + h * DH, k_ok, hh);
  store_rows<DH>(dva, 1.0f, p.dv + tok_row * p.dvs + h * DH, k_ok, hh);
}

// Both roles in one launch: each alone is bound by the chain of its longest workgroup (a wave walks the
// tokens of its image).  Workgroup -> (xcd = id % 8, number inside the XCD): first the dkdv blocks, longest image
// first (live_order), then the dq blocks in the same order: alternating roles would give every other unit only
// the longer of the two.  Waves of longer images run at a higher priority, as the launch ends with them.
// Bound by vector instructions and the waits between them: per 32 x 32 block the two roles issue 14 MFMAs (448
// cycles) and about 125 vector instructions, 32 of them exponentials (630 cycles), at three (head dim 64: two)
// wavefronts per SIMD; a fourth, without the second score block in flight, is 2-8 % faster on launches of several
// rounds and 10-25 % slower on smaller ones.  No load is waited for between two tiles (see PairStage).
// 16 images of 3136 tokens, 10-60 % selected, 3 heads of 32: 74 -> 52 us; 32 x 1024 tokens, all selected, 12
// heads of 64: 508 -> 410 us; 2 x 4200 tokens, 5-40 %, 8 heads of 32: 28 -> 20 us; 122 x 480 tokens, 6-48 %, 11 heads
// of 64, where every workgroup ranked the segments in LDS and those without a block lay between the others: 267 -> 160.
template <int DH, int MODE>
__device__ __forceinline__ void bwd_long_block(const BwdArgs& p, unsigned block, unsigned blocks) {
  __shared__ BwdLongLds<DH> lds;
  __shared__ LiveTile s_live;
  const int xcd = block & 7, jj = block >> 3, half = blocks >> 4, nblk = p.nblk;
  Segment seg = {0, 0, 0};
  int h = 0, r0 = 0;
  bool dkdv;
  if (p.B <= kLptMaxB) {
    const LiveTile lt = live_tiles_apply(p.H, p.B)
                            ? live_tile_block<2>(xcd, jj, p.H, p.B, p.cu, kBwdRows, nblk, &s_live)
                            : class_tile_block<2>(xcd, jj, p.H, p.B, p.cu, kBwdRows, nblk, &s_live);
    if (lt.valid) seg = {lt.row0, lt.len, lt.len};
    h = lt.h;
    r0 = lt.qb * kBwdRows;
    dkdv = !lt.again;
    const int weight = dkdv ? 3 * lt.len : 2 * lt.len;
    if (weight > 2 * lt.longest) __builtin_amdgcn_s_setprio(2);
    else if (weight > lt.longest) __builtin_amdgcn_s_setprio(1);
  } else {
    dkdv = jj < half;
    const TileId t = xcd_tile_at(xcd, dkdv ? jj : jj - half, nblk, p.H, p.B);
    if (t.valid) seg = segment_of(t.rank, p.cu, nullptr, 0);
    h = t.h;
    r0 = t.qb * kBwdRows;
  }
  if (r0 < seg.nk) {
    if (dkdv) bwd_dkdv_role<DH, MODE, false>(lds, p, seg, h, r0);
    else bwd_dq_role<DH, MODE, false>(lds, p, seg, h, r0);
  }
  __builtin_amdgcn_s_setprio(0);
  if (MODE != kPacked) {
    // gradients of the unselected tokens: every workgroup (with or without a tile) zeroes an even share of the
    // rows, a quarter per wave
    constexpr int NW = kBwdThreads / 64;
    const long units = (long)blocks * NW, u = (long)block * NW + (threadIdx.x >> 6);
    const long per = (p.tok.rows + units - 1) / units, z0 = min(p.tok.rows, u * per), z1 = min(p.tok.rows, z0 + per);
    const int lane = threadIdx.x & 63;
    zero_unselected_rows(p.dq, p.dqs, p.H * DH, p.tok.inv_pos, z0, z1, lane);
    zero_unselected_rows(p.dk, p.dks, p.H * DH, p.tok.inv_pos, z0, z1, lane);
    zero_unselected_rows(p.dv, p.dvs, p.H * DH, p.tok.inv_pos, z0, z1, lane);
  }
}

// The same for calls of up to 64 segments and 512 (segment, head) pairs in a launch group, or with segments of up to 4
// blocks: at most as many workgroups as are resident together, of which number g of an XCD's G takes blocks g, 2 G - 1 - g,
// 2 G + g, ... of the order.  A grid with a workgroup for each block of the longest possible segments puts
// thousands without a block, 3.5 us of a slot each, in front of the next call's (four stages of 16 images, 3136 to
// 49 tokens: 2868 of 5280; the step 163 -> 156 us; 64 x 400 tokens, 6 heads of 64: 115 -> 112).  Long segments in a
// launch of their own end with them, and are better dealt as slots become free (4 x 4200 tokens, 8 heads of 32: 91.6 against 93.0
// us; 32 x 3136: 340 against 347).
constexpr int bwd_long_slots(int DH) { return (DH == 32 ? 3 : 2) * 256; }
template <int DH, int MODE>
__device__ __forceinline__ void bwd_resident_block(const BwdArgs& p, unsigned block, unsigned blocks) {
  __shared__ BwdLongLds<DH> lds;
  __shared__ int s_order[5][64];
  const int xcd = block & 7, G = blocks >> 3, g = there_and_back(block >> 3, G), lane = threadIdx.x & 63;
  if (threadIdx.x < 64) {
    const LiveOrder o = live_order(xcd, p.H, p.B, p.cu, kBwdRows, p.nblk);
    s_order[0][lane] = o.len;
    s_order[1][lane] = o.start;
    s_order[2][lane] = o.img;
    s_order[3][lane] = o.nb;
    s_order[4][lane] = o.incl;
  }
  __syncthreads();
  for (int round = 0;; ++round) {
    const LiveOrder o = {s_order[0][lane], s_order[1][lane], s_order[2][lane], s_order[3][lane], s_order[4][lane]};
    const LiveTile lt = live_pick<2>(o, xcd, round * G + (round & 1 ? G - 1 - g : g), p.H);
    if (!lt.valid) break;
    if (round > 0) __syncthreads();                  // every wave is past its last read of the tiles
    const Segment seg = {lt.row0, lt.len, lt.len};
    if (!lt.again) bwd_dkdv_role<DH, MODE, true>(lds, p, seg, lt.h, lt.qb * kBwdRows);
    else bwd_dq_role<DH, MODE, true>(lds, p, seg, lt.h, lt.qb * kBwdRows);
  }
  if (MODE != kPacked) {
    // gradients of the unselected tokens: zeroed by the workgroups without a block, which run beside the others, or by
    // all where those are few; an even share of the XCD's eighth of the rows each, a quarter per wave
    constexpr int NW = kBwdThreads / 64;
    const int busy = min(G, 2 * __builtin_amdgcn_readfirstlane(s_order[4][63])), idle = G - busy;
    const bool by_idle = 4 * idle >= G;
    if (by_idle && g < busy) return;
    const long from = p.tok.rows * xcd / 8, to = p.tok.rows * (xcd + 1) / 8;
    const long units = (long)(by_idle ? idle : G) * NW, u = (long)(by_idle ? g - busy : g) * NW + (threadIdx.x >> 6);
    const long per = (to - from + units - 1) / units, z0 = min(to, from + u * per), z1 = min(to, z0 + per);
    zero_unselected_rows(p.dq, p.dqs, p.H * DH, p.tok.inv_pos, z0, z1, lane);
    zero_unselected_rows(p.dk, p.dks, p.H * DH, p.tok.inv_pos, z0, z1, lane);
    zero_unselected_rows(p.dv, p.dvs, p.H * DH, p.tok.inv_pos, z0, z1, lane);
  }
}

template <int DH, int MODE>
__global__ void __launch_bounds__(kBwdThreads) __attribute__((amdgpu_waves_per_eu(DH == 32 ? 3 : 2)))
attn_bwd_long_bf16_kernel(const BwdArgs p) {
  bwd_long_block<DH, MODE>(p, blockIdx.x, gridDim.x);
}
template <int DH, int MODE>
__global__ void __launch_bounds__(kBwdThreads) __attribute__((amdgpu_waves_per_eu(DH == 32 ? 3 : 2)))
attn_bwd_resident_bf16_kernel(const BwdArgs p) {
  bwd_resident_block<DH, MODE>(p, blockIdx.x, gridDim.x);
}

// D[h][j] = <dO_j, O_j> over head h's columns, for the packed rows j < cu[B]: DH / 8 adjacent
// lanes share a (row, head).  A launch of 4 to 6 us for a few MB; where dO is known before the forward pass, that pass forms
// D with the same sums from the rows it holds (fwd_flush), and this launch falls away.  us a training step: 32 x 400 tokens, 6
// heads of 64, 64.6 -> 61.6, 12 x 720, 8 heads of 32, 45.0 -> 42.1, 8 x 1024, 12 heads of 64, 94.3 -> 91.1; four stages of 16 x 3136
// tokens as launch groups 136.8 -> 133.7, of one image 62.9 -> 60.3.
template <int DH>
__device__ __forceinline__ void bwd_dvec_block(const BwdArgs& p, unsigned block, unsigned blocks) {
  constexpr int CPR = DH / 8;
  const int H = p.H;
  const int32_t* gather_idx = p.tok.gather_idx;
  const long C = (long)H * DH, total = (long)p.cu[p.B] * H * CPR;
  for (long i = (long)block * 256 + threadIdx.x; i < ((total + 63) & ~63L); i += (long)blocks * 256) {
    const long rh = i / CPR;
    const int c = (int)(i % CPR);
    const long row = rh / H;
    const int h = (int)(rh % H);
    float d = 0.f;
    if (i < total) {
      const floatx8 of = bf16x8_to_float(*reinterpret_cast<const bf16x8*>(p.out + row * C + h * DH + c * 8));
      const long grow = gather_idx != nullptr ? (long)gather_idx[row] : row;
      const floatx8 gf = bf16x8_to_float(*reinterpret_cast<const bf16x8*>(p.dout + grow * C + h * DH + c * 8));
#pragma unroll
      for (int e = 0; e < 8; ++e) d = fmaf(of[e], gf[e], d);
    }
    d = adjacent_sum<CPR>(d);
    if (i < total && c == 0) p.dvec[h * p.lse_stride + row] = d;
  }
}
template <int DH>
__global__ void __launch_bounds__(256) attn_bwd_dvec_kernel(const BwdArgs p) {
  bwd_dvec_block<DH>(p, blockIdx.x, gridDim.x);
}
static unsigned dvec_blocks(long rows, int H, int Dh) { return (unsigned)std::min<long>((rows * H * (Dh / 8) + 255) / 256, 4096L); }
void launch_dvec(const void* out, const void* dy, const int32_t* gather_idx, const int32_t* cu, int B, int H, int Dh, long lse_stride,
                 float* dvec, hipStream_t st) {
  BwdArgs args = {};
  args.out = static_cast<const __bf16*>(out);
  args.dout = static_cast<const __bf16*>(dy);
  args.tok.gather_idx = gather_idx;
  args.cu = cu;
  args.B = B;
  args.H = H;
  args.lse_stride = lse_stride;
  args.dvec = dvec;
  const dim3 grid(dvec_blocks(lse_stride, H, Dh));
  if (Dh == 32) hipLaunchKernelGGL((attn_bwd_dvec_kernel<32>), grid, dim3(256), 0, st, args);
  else hipLaunchKernelGGL((attn_bwd_dvec_kernel<64>), grid, dim3(256), 0, st, args);
}

// Several calls in one launch (launch groups, head dim 32, gradients at token positions): whatever the segment
// lengths, the long-segment form (the short one's workgroups have the size of their segments).
__global__ void __launch_bounds__(256) attn_bwd_dvec_group_kernel(const Members<BwdArgs> m) {
  const MemberBlock mb = member_of(m, blockIdx.x);
  bwd_dvec_block<32>(m.a[mb.s], mb.block, mb.blocks);
}
template <int MODE, bool RESIDENT>
__global__ void __launch_bounds__(kBwdThreads) __attribute__((amdgpu_waves_per_eu(3)))
attn_bwd_group_kernel(const Members<BwdArgs> m) {
  const MemberBlock mb = member_of(m, blockIdx.x);
  if (RESIDENT) {
    const BwdArgs a = m.a[mb.s];
    bwd_resident_block<32, MODE>(a, mb.block, mb.blocks);
  } else bwd_long_block<32, MODE>(m.a[mb.s], mb.block, mb.blocks);
}
static thread_local Noted<BwdArgs> g_noted[2], g_noted_dvec[2];      // packed, gated operands
void group_forget_attention_bwd() { g_noted[0].n = g_noted[1].n = g_noted_dvec[0].n = g_noted_dvec[1].n = 0; }
template <int MODE>
static void flush_mode(hipStream_t st) {
  constexpr int g = MODE == kGated;
  if (g_noted[g].n == 0) return;
  Members<BwdArgs> m;
  if (g_noted_dvec[g].n > 0) {
    const unsigned dblocks = g_noted_dvec[g].members(m);
    hipLaunchKernelGGL(attn_bwd_dvec_group_kernel, dim3(dblocks), dim3(256), 0, st, m);
  }
  bool resident = true;
  for (int i = 0; i < g_noted[g].n; ++i) resident = resident && live_tiles_apply(g_noted[g].a[i].H, g_noted[g].a[i].B);
  for (int i = 0; resident && i < g_noted[g].n; ++i)
    g_noted[g].blocks[i] = std::min(g_noted[g].blocks[i], (unsigned)bwd_long_slots(32));
  const unsigned blocks = g_noted[g].members(m);
  if (resident) hipLaunchKernelGGL((attn_bwd_group_kernel<MODE, true>), dim3(blocks), dim3(kBwdThreads), 0, st, m);
  else hipLaunchKernelGGL((attn_bwd_group_kernel<MODE, false>), dim3(blocks), dim3(kBwdThreads), 0, st, m);
}
int group_flush_attention_bwd(hipStream_t st) {
  flush_mode<kTokens>(st);
  flush_mode<kGated>(st);
  return check_launch("spa_group_end");
}

// ------------------------------------------------- dQ, dK, dV in one kernel (short segments)
// One workgroup per (image, head), one wave per 32 tokens of the longest segment; wave j owns the
// segment's tokens 32j .. 32j+31, first as keys, then as queries.
//   keys:    Q and dO of the segment in LDS; S = Q_t K_j^T (a lane holds 16 queries of ONE key), then
//            dV_j^T += dO_t^T P and, with dP = dO_t V_j^T, dK_j^T += Q_t^T dS over the query tiles t;
//   queries: K and V of the segment, from the registers of the waves that own them, in the same LDS;
//            S^T = K_t Q_j^T, dP^T = V_t dO_j^T (16 keys of one query in a lane), dQ_j^T += K_t^T dS^T over
//            the key tiles t.
// S (and at head dim 64 P, see kOnePass) is computed again instead of exchanged: no dS tiles, no dQ
// accumulators in LDS, no barrier inside either half, so the waves of a workgroup drift apart, and with
// 65 instead of 141 KB at 196 tokens and at most 128 registers two workgroups share a unit: one loads
// while the other multiplies.  No atomics, every sum in a fixed order: run-to-run bit-stable.
// Measured on the ViT-B-shaped batch (64 x 196 tokens, 12 heads of 64): 44.8 -> 37.3 us; 128 images, their order by
// ballots instead of a ranking in LDS in every workgroup: 82 -> 72.  Bound by its memory phases: without any walk it takes 26 of
// 36 us (77 MB of rows, 29 MB of zeros), so the K and V rows are not fetched a second time: 40.0 -> 36.2 us (q, k, v
// at token positions), 128 images with packed rows 61 -> 51.6.  Two short segments in one workgroup, so that all its waves
// have tokens: 38.1 | 38.0 us with | without, 128 images 52.7 | 52.1 - fewer workgroups overlap their phases less.
// Operand rows: packed (row0 + j), or GATED: q, k, v at token positions (row gather_idx[j]), the v row
// multiplied by Sigmoid(score) and rounded to bf16 (r_g = Sigmoid(s) . r, as a packed r_g holds it).
// Dynamic LDS, rows = 32 * nw:  A [rows][DH+8] (Q, then K) | B [rows][DH+8] (dO, then V) |
// lse*log2(e) [rows] | D [rows].
template <int DH>
__host__ __device__ constexpr size_t bwd_short_lds_bytes(int nw) {
  return (size_t)nw * (2 * 32 * (DH + 8) * 2 + 2 * 32 * 4);
}

// Heaviest image first, but the second workgroup of every unit takes the lightest images: the first 512 workgroups start together, and
// with images of like length they all load, then all multiply, then all store.  Where two workgroups share a unit (six waves or more)
// and from 832 (image, head) pairs on; us a training step, by weight alone | so, heads of 64: 64 x 196 tokens, 12 heads (768 pairs) 82.1 | 82.3, 72 images 98.2 | 97.7,
// 80 106.4 | 103.9, 128 154.4 | 152.7, 64 of 16 heads 105.8 | 102.1, 110 x 169, 12 heads 127.7 | 124.1; 48 x 196 (576 pairs) 68.5 |
// 73.8; 96 x 100, where four share a unit, 75.6 | 77.1; heads of 32, 100 x 196 85.9 | 86.3.
__device__ __forceinline__ int staggered_place(int rank, int B, int H) {
  const int first = 256 / H;                         // images of the first workgroup of every unit
  return rank < first ? rank : rank < 2 * first ? B - 1 - (rank - first) : rank - first;
}

template <int DH, bool GATED>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
attn_bwd_short_bf16_kernel(const BwdArgs p) {
  constexpr int RS = DH + 8, KK = DH / 16, DB = DH / 32, CPR = DH / 8, PER = CPR / 2;
  constexpr bool kOnePass = DH == 32;                // dV and dK in one walk (at 64 their accumulators and operands need 150 registers)
  extern __shared__ __attribute__((aligned(16))) unsigned char bwd_smem[];
  const int threads = blockDim.x, nw = threads >> 6, rows_cap = 32 * nw;
  __bf16* As = reinterpret_cast<__bf16*>(bwd_smem);
  __bf16* Bs = As + rows_cap * RS;
  float* lse2s = reinterpret_cast<float*>(Bs + rows_cap * RS);
  float* Ds = lse2s + rows_cap;

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, l32 = lane & 31, hh = lane >> 5;
  const int H = p.H, B = p.B, h = blockIdx.x % H, rank = blockIdx.x / H;
  const int32_t* cu = p.cu;
  const bool at_tokens = p.tok.gather_idx != nullptr;
  // by weight (work per segment grows like n^2)
  int img = rank, start = 0, len = 0;
  if (B > 1 && B <= 8 * kWave) {                     // every wave ranks on its own: no LDS, no barrier
    const int place = DH == 64 && nw >= 6 && (long)B * H >= 832 ? staggered_place(rank, B, H) : rank;
    const RankedSegment rs = B <= kWave       ? ranked_segment_wave<1>(place, B, cu, nw)
                             : B <= 2 * kWave ? ranked_segment_wave<2>(place, B, cu, nw)
                                              : ranked_segment_wave<8>(place, B, cu, nw);
    img = rs.img;
    start = rs.row0;
    len = rs.len;
  } else {                                           // (more images: in index order)
    start = cu[img];
    len = cu[img + 1] - start;
  }
  const long row0 = start;
  const int n = min(len, rows_cap);
  if (n > 0) {
    const int nws = (n + 31) >> 5;                   // waves with tokens = tiles
    const long C = (long)H * DH;
    const float scale_log2 = p.scale * kLog2e;
    const int32_t* gi = at_tokens ? p.tok.gather_idx + row0 : nullptr;
    auto token_row = [&](int r) { return at_tokens ? (long)gi[r] : row0 + r; };   // where dO and the gradients live
    auto src_row = [&](int r) { return GATED ? (long)gi[r] : row0 + r; };         // where q, k, v live

    // ---- Q, dO into LDS (every thread PER chunks of each), D_i = <dO_i, O_i>, lse_i; wave j: K_j, V_j
    {
      bf16x8 qreg[PER], greg[PER], oreg[PER];
      float lreg[PER];
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        const int i = tid + t * threads, r = i / CPR, c = i % CPR;
        qreg[t] = zero_bf16x8(); greg[t] = zero_bf16x8(); oreg[t] = zero_bf16x8();
        lreg[t] = INFINITY;                          // rows past the segment: probability 0
        if (r < n) {
          qreg[t] = *reinterpret_cast<const bf16x8*>(p.q + src_row(r) * p.qs + h * DH + c * 8);
          greg[t] = *reinterpret_cast<const bf16x8*>(p.dout + token_row(r) * C + h * DH + c * 8);
          oreg[t] = *reinterpret_cast<const bf16x8*>(p.out + (row0 + r) * C + h * DH + c * 8);
          if (c == 0) lreg[t] = p.lse[h * p.lse_stride + row0 + r] * kLog2e;
        }
      }
#pragma unroll
      for (int t = 0; t < PER; ++t) {
        const int i = tid + t * threads, r = i / CPR, c = i % CPR;
        *reinterpret_cast<bf16x8*>(&As[r * RS + c * 8]) = qreg[t];
        *reinterpret_cast<bf16x8*>(&Bs[r * RS + c * 8]) = greg[t];
        const floatx8 gf = bf16x8_to_float(greg[t]), of = bf16x8_to_float(oreg[t]);
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) d = fmaf(of[e], gf[e], d);
        d = adjacent_sum<CPR>(d);                                           // the CPR chunks of a row: adjacent lanes
        if (c == 0) {
          Ds[r] = d;
          lse2s[r] = lreg[t];
        }
      }
    }
    const bool live = wv < nws;
    const int ti = wv * 32 + l32;                    // this lane's token, as key and as query
    const bool t_ok = ti < n;
    const long my_src = t_ok ? src_row(ti) : 0, my_row = t_ok ? token_row(ti) : 0;
    const float my_gate = GATED && t_ok ? sigmoidf_dev(p.v_scores[my_src]) : 1.f;
    bf16x8 kf[KK], vf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      kf[kk] = zero_bf16x8();
      vf[kk] = zero_bf16x8();
      if (t_ok) {
        const int col = h * DH + kk * 16 + hh * 8;
        kf[kk] = *reinterpret_cast<const bf16x8*>(p.k + my_src * p.ks + col);
        vf[kk] = *reinterpret_cast<const bf16x8*>(p.v + my_src * p.vs + col);
        if (GATED) vf[kk] = scale_row(vf[kk], my_gate);
      }
    }
    __syncthreads();

    // ---- as keys
    if (live) {
      floatx16 dka[DB], dva[DB];
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dka[d][r] = 0.f; dva[d][r] = 0.f; }
      auto walk = [&](auto want_dv, auto want_dk) {
        constexpr bool kDv = decltype(want_dv)::value, kDk = decltype(want_dk)::value;
        for (int t = 0; t < nws; ++t) {
          const __bf16* Qt = As + t * 32 * RS;
          const __bf16* Gt = Bs + t * 32 * RS;
          floatx16 s, dp;
#pragma unroll
          for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; }
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            const bf16x8 qa = *reinterpret_cast<const bf16x8*>(&Qt[l32 * RS + kk * 16 + hh * 8]);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa, kf[kk], s, 0, 0, 0);
            if (kDk) {
              const bf16x8 ga = *reinterpret_cast<const bf16x8*>(&Gt[l32 * RS + kk * 16 + hh * 8]);
              dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ga, vf[kk], dp, 0, 0, 0);
            }
          }
#pragma unroll
          for (int mf = 0; mf < 2; ++mf) {
            floatx8 fp, fd;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
              const int at = t * 32 + 16 * mf + 8 * g + 4 * hh;
              const floatx4 l4 = *reinterpret_cast<const floatx4*>(&lse2s[at]);
              const floatx4 d4 = *reinterpret_cast<const floatx4*>(&Ds[at]);
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const int i = 8 * mf + 4 * g + e;
                fp[4 * g + e] = __builtin_amdgcn_exp2f(fmaf(s[i], scale_log2, -l4[e]));
                if (kDk) fd[4 * g + e] = fp[4 * g + e] * (dp[i] - d4[e]);
              }
            }
            if (kDv) {
              const bf16x8 pb = float_to_bf16x8(fp);
#pragma unroll
              for (int d = 0; d < DB; ++d)
                dva[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(transposed_frag_rowmajor<RS>(Gt, d, 0, mf, lane), pb, dva[d], 0, 0, 0);
            }
            if (kDk) {
              const bf16x8 dsb = float_to_bf16x8(fd);
#pragma unroll
              for (int d = 0; d < DB; ++d)
                dka[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(transposed_frag_rowmajor<RS>(Qt, d, 0, mf, lane), dsb, dka[d], 0, 0, 0);
            }
          }
        }
      };
      if constexpr (kOnePass) {
        walk(std::true_type{}, std::true_type{});
        store_rows<DH>(dva, 1.0f, p.dv + my_row * p.dvs + h * DH, t_ok, hh);
      } else {
        walk(std::true_type{}, std::false_type{});
        store_rows<DH>(dva, 1.0f, p.dv + my_row * p.dvs + h * DH, t_ok, hh);
        walk(std::false_type{}, std::true_type{});
      }
      store_rows<DH>(dka, p.scale, p.dk + my_row * p.dks + h * DH, t_ok, hh);
    }

    // ---- as queries: Q_j, dO_j from LDS to registers, then every wave's K and V rows, which it holds, take their place
    bf16x8 qf[KK], gf[KK];
    float D = 0.f, lse2 = INFINITY;                  // (queries past the segment: probability 0)
    if (live) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        qf[kk] = *reinterpret_cast<const bf16x8*>(&As[ti * RS + kk * 16 + hh * 8]);
        gf[kk] = *reinterpret_cast<const bf16x8*>(&Bs[ti * RS + kk * 16 + hh * 8]);
      }
      D = Ds[ti];
      lse2 = lse2s[ti];
    }
    __syncthreads();                                 // every wave is done with Q and dO
    if (live) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        *reinterpret_cast<bf16x8*>(&As[ti * RS + kk * 16 + hh * 8]) = kf[kk];
        *reinterpret_cast<bf16x8*>(&Bs[ti * RS + kk * 16 + hh * 8]) = vf[kk];
      }
    }
    __syncthreads();
    if (live) {
      floatx16 acc[DB];
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[d][r] = 0.f;
      for (int t = 0; t < nws; ++t) {
        const __bf16* Kt = As + t * 32 * RS;
        const __bf16* Vt = Bs + t * 32 * RS;
        floatx16 s, dp;
#pragma unroll
        for (int e = 0; e < 16; ++e) { s[e] = 0.f; dp[e] = 0.f; }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const bf16x8 ka = *reinterpret_cast<const bf16x8*>(&Kt[l32 * RS + kk * 16 + hh * 8]);
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, qf[kk], s, 0, 0, 0);
          const bf16x8 va = *reinterpret_cast<const bf16x8*>(&Vt[l32 * RS + kk * 16 + hh * 8]);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, gf[kk], dp, 0, 0, 0);
        }
        const int left = n - t * 32;                 // valid keys of the tile
        if (left < 32) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (acc_row(r, hh) >= left) s[r] = -INFINITY;
        }
#pragma unroll
        for (int mf = 0; mf < 2; ++mf) {
          floatx8 f;
#pragma unroll
          for (int j = 0; j < 8; ++j)
            f[j] = __builtin_amdgcn_exp2f(fmaf(s[8 * mf + j], scale_log2, -lse2)) * (dp[8 * mf + j] - D);
          const bf16x8 dsb = float_to_bf16x8(f);
#pragma unroll
          for (int d = 0; d < DB; ++d)
            acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(transposed_frag_rowmajor<RS>(Kt, d, 0, mf, lane), dsb, acc[d], 0, 0, 0);
        }
      }
      store_rows<DH>(acc, p.scale, p.dq + my_row * p.dqs + h * DH, t_ok, hh);
    }
  }
  // this head's columns of the unselected rows of this workgroup's share (last: nothing waits for them)
  if (at_tokens) {
    const long per = (p.tok.rows + B - 1) / B, i0 = rank * per, i1 = min(p.tok.rows, i0 + per);
    const bf16x8 z = zero_bf16x8();
    for (long i = i0 * CPR + tid; i < i1 * CPR; i += threads) {
      const long row = i / CPR;
      const int c = (int)(i % CPR);
      if (p.tok.inv_pos[row] < 0) {
        *reinterpret_cast<bf16x8*>(p.dq + row * p.dqs + h * DH + c * 8) = z;
        *reinterpret_cast<bf16x8*>(p.dk + row * p.dks + h * DH + c * 8) = z;
        *reinterpret_cast<bf16x8*>(p.dv + row * p.dvs + h * DH + c * 8) = z;
      }
    }
  }
}

// ------------------------------------------------------------------------------- fp32
// One thread per row (a query for dQ, a key for dK/dV); the other side streams through LDS.
// kKeySide = false: rows are queries, outputs dq (and D_i).  true: rows are keys, outputs dk, dv.
template <int DH, bool kKeySide>
__global__ void __launch_bounds__(128)
attn_bwd_f32_kernel(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                    long qs, long ks, long vs, const float* __restrict__ out, const float* __restrict__ dout,
                    const float* __restrict__ lse, float* __restrict__ dvec, long lse_stride,
                    const int32_t* __restrict__ cu, int H, float scale, float* __restrict__ g0, long g0s,
                    float* __restrict__ g1, long g1s, TokenIO tok) {
  constexpr int BM = 128, BN = 32;
  __shared__ __attribute__((aligned(16))) float As[BN * DH];   // K (query side) or Q (key side)
  __shared__ __attribute__((aligned(16))) float Bs[BN * DH];   // V (query side) or dO (key side)
  __shared__ float lses[BN], Dss[BN];

  const int h = blockIdx.y;
  const Seg seg = seg_of(blockIdx.z, cu);
  const int r0 = blockIdx.x * BM;
  const int tid = threadIdx.x;
  const bool at_tokens = tok.gather_idx != nullptr;
  if (at_tokens) {   // gradients of the unselected tokens: this head's columns of an even share of the rows
    const long units = (long)gridDim.x * gridDim.z, u = (long)blockIdx.z * gridDim.x + blockIdx.x;
    const long per = (tok.rows + units - 1) / units, i0 = min(tok.rows, u * per), i1 = min(tok.rows, i0 + per);
    const floatx4 z = {0.f, 0.f, 0.f, 0.f};
    for (long i = i0 * (DH / 4) + tid; i < i1 * (DH / 4); i += BM) {
      const long row = i / (DH / 4);
      const int c = (int)(i % (DH / 4));
      if (tok.inv_pos[row] < 0) {
        *reinterpret_cast<floatx4*>(g0 + row * g0s + h * DH + c * 4) = z;
        if (kKeySide) *reinterpret_cast<floatx4*>(g1 + row * g1s + h * DH + c * 4) = z;
      }
    }
  }
  if (r0 >= seg.n) return;
  const int ri = r0 + tid;
  const bool ok = ri < seg.n;
  const long C = (long)H * DH;
  const long grow = seg.row0 + ri;
  const long trow = ok && at_tokens ? (long)tok.gather_idx[grow] : grow;   // where this row's gradients live

  float a[DH], b[DH], acc0[DH], acc1[DH];
#pragma unroll
  for (int d = 0; d < DH; ++d) { a[d] = 0.f; b[d] = 0.f; acc0[d] = 0.f; acc1[d] = 0.f; }
  float my_lse = 0.f, my_D = 0.f;
  if (ok) {
    if (!kKeySide) {
      float dsum = 0.f;
#pragma unroll
      for (int d = 0; d < DH; ++d) {
        a[d] = q[grow * qs + h * DH + d];
        b[d] = dout[trow * C + h * DH + d];
        dsum = fmaf(b[d], out[grow * C + h * DH + d], dsum);
      }
      my_D = dsum;
      my_lse = lse[h * lse_stride + grow];
      dvec[h * lse_stride + grow] = dsum;
    } else {
#pragma unroll
      for (int d = 0; d < DH; ++d) {
        a[d] = k[grow * ks + h * DH + d];
        b[d] = v[grow * vs + h * DH + d];
      }
    }
  }
  const float* sa = kKeySide ? q : k;
  const float* sb = kKeySide ? dout : v;
  const long sa_stride = kKeySide ? qs : ks;
  const long sb_stride = kKeySide ? C : vs;

  for (int t = 0; t < seg.n; t += BN) {
    __syncthreads();
    for (int i = tid; i < BN * DH / 4; i += BM) {
      const int r = i / (DH / 4), c = i % (DH / 4);
      floatx4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
      if (t + r < seg.n) {
        const long prow = seg.row0 + t + r;
        const long brow = kKeySide && at_tokens ? (long)tok.gather_idx[prow] : prow;   // dO rows sit at the tokens
        x = *reinterpret_cast<const floatx4*>(sa + prow * sa_stride + h * DH + c * 4);
        y = *reinterpret_cast<const floatx4*>(sb + brow * sb_stride + h * DH + c * 4);
      }
      *reinterpret_cast<floatx4*>(&As[r * DH + c * 4]) = x;
      *reinterpret_cast<floatx4*>(&Bs[r * DH + c * 4]) = y;
    }
    if (kKeySide && tid < BN) {
      const bool in = t + tid < seg.n;
      lses[tid] = in ? lse[h * lse_stride + seg.row0 + t + tid] : INFINITY;
      Dss[tid] = in ? dvec[h * lse_stride + seg.row0 + t + tid] : 0.f;
    }
    __syncthreads();
    const int tn = min(BN, seg.n - t);
    for (int j = 0; j < tn; ++j) {
      float s = 0.f, dp = 0.f;
#pragma unroll
      for (int d = 0; d < DH; ++d) {
        s = fmaf(a[d], As[j * DH + d], s);     // q.k
        dp = fmaf(b[d], Bs[j * DH + d], dp);   // dO.v
      }
      const float l = kKeySide ? lses[j] : my_lse;
      const float D = kKeySide ? Dss[j] : my_D;
      const float p = expf(s * scale - l);
      const float ds = p * (dp - D) * scale;
#pragma unroll
      for (int d = 0; d < DH; ++d) {
        acc0[d] = fmaf(ds, As[j * DH + d], acc0[d]);              // dq += ds k   | dk += ds q
        if (kKeySide) acc1[d] = fmaf(p, Bs[j * DH + d], acc1[d]);  //              | dv += p dO
      }
    }
  }
  if (!ok) return;
#pragma unroll
  for (int d = 0; d < DH; ++d) {
    g0[trow * g0s + h * DH + d] = acc0[d];
    if (kKeySide) g1[trow * g1s + h * DH + d] = acc1[d];
  }
}

}  // namespace spa

using namespace spa;

extern "C" size_t spa_attention_bwd_workspace_bytes(int B, int max_seqlen, int H, int Dh, int dtype) {
  (void)Dh; (void)dtype;
  if (B < 1 || max_seqlen < 1 || H < 1) return 0;
  return (size_t)H * (size_t)B * (size_t)max_seqlen * sizeof(float);   // D_i for every (head, row)
}

// Short segments whose (image, head) pairs, one workgroup each in the one-kernel form, leave most of the 256 units
// idle take the long-segment form, whose roles and 128-row blocks are workgroups of their own.  It costs a launch more
// (D), which the smallest segments and batches do not earn back: us of the training step, one kernel -> long form,
// 196 tokens, head dim 64: 12 pairs +0.9, 24 -4.4, 96 -3.7, 252 -3.2, 384 +0.1; 49 tokens: 24 +0.4, 252 -1.0; head dim
// 32, 196 tokens: 24 +0.7, 48 -0.6, 192 -2.0, 252 -0.6, 384 +2.4; 144 tokens: no gain.
static bool few_pairs(int B, int H, int Dh, int n_max) {
  const long pairs = (long)B * H;
  return B > 1 && B <= kWave && (Dh == 64 ? n_max > 64 && pairs >= 16 && pairs <= 288 : n_max > 160 && pairs >= 32 && pairs <= 256);
}

// tok.gather_idx != nullptr: gradients in and out at token positions.  spread: few_pairs decides, where the caller
// gave the workspace.
static int attention_bwd_common(const char* fn, const void* q, const void* k, const void* v, int64_t q_row_stride,
                                int64_t k_row_stride, int64_t v_row_stride, const void* out, const void* dout,
                                const float* lse, const int32_t* cu_seqlens, int B, int max_seqlen, int H, int Dh,
                                int dtype, float softmax_scale, void* dq, void* dk, void* dv,
                                int64_t dq_row_stride, int64_t dk_row_stride, int64_t dv_row_stride,
                                void* workspace, size_t workspace_bytes, TokenIO tok, void* stream,
                                bool spread, const float* v_scores = nullptr, bool have_d = false) {
  const bool at_tokens = tok.gather_idx != nullptr;
  SPA_REQUIRE(q && k && v && out && dout && lse && cu_seqlens && dq && dk && dv, SPA_ERR_INVALID_ARG,
              "%s: null pointer", fn);
  SPA_REQUIRE(B >= 1 && max_seqlen >= 1 && H >= 1, SPA_ERR_INVALID_ARG, "%s: B, max_seqlen, H must be >= 1", fn);
  SPA_REQUIRE((long)B * max_seqlen < 2147483647L, SPA_ERR_INVALID_ARG, "%s: B*max_seqlen must be < 2^31", fn);
  SPA_REQUIRE(B <= 65535 && H <= 65535, SPA_ERR_INVALID_ARG, "%s: B and H must be <= 65535", fn);
  SPA_REQUIRE(dtype == SPA_F32 || dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: unknown dtype %d", fn, dtype);
  SPA_REQUIRE(Dh == 32 || Dh == 64, SPA_ERR_UNSUPPORTED, "%s: head dim %d not supported (32 or 64)", fn, Dh);
  const int64_t strides[6] = {q_row_stride, k_row_stride, v_row_stride, dq_row_stride, dk_row_stride, dv_row_stride};
  for (int64_t rs : strides) {
    SPA_REQUIRE(rs >= (int64_t)H * Dh, SPA_ERR_INVALID_ARG, "%s: row stride %ld < H*Dh", fn, (long)rs);
    SPA_REQUIRE((rs * elem_size(dtype)) % 16 == 0, SPA_ERR_INVALID_ARG, "%s: row strides must be multiples of 16 bytes", fn);
  }
  SPA_REQUIRE(aligned16(q) && aligned16(k) && aligned16(v) && aligned16(out) && aligned16(dout) &&
                  aligned16(dq) && aligned16(dk) && aligned16(dv),
              SPA_ERR_INVALID_ARG, "%s: tensors not 16-byte aligned", fn);
  SPA_REQUIRE(softmax_scale >= 0.f && std::isfinite(softmax_scale), SPA_ERR_INVALID_ARG,
              "%s: softmax_scale must be finite and >= 0", fn);
  // short segments: the one-kernel form, which needs no workspace (option attn_bwd_short = "tiled" takes the
  // long-segment kernel)
  const size_t dvec_bytes = spa_attention_bwd_workspace_bytes(B, max_seqlen, H, Dh, dtype);
  const bool short_seg = max_seqlen <= 256 && !options().bwd_tiled && !group_open() &&
                         !(spread && few_pairs(B, H, Dh, max_seqlen) && workspace != nullptr && workspace_bytes >= dvec_bytes);
  const bool one_kernel = dtype == SPA_BF16 && short_seg;
  const size_t need = one_kernel ? 0 : dvec_bytes;
  SPA_REQUIRE(need == 0 || (workspace != nullptr && workspace_bytes >= need), SPA_ERR_WORKSPACE,
              "%s: workspace of %zu bytes needed, %zu given", fn, need, workspace_bytes);
  const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt((float)Dh);
  const long ls = (long)B * max_seqlen;
  float* dvec = static_cast<float*>(workspace);
  hipStream_t st = as_stream(stream);
  SPA_REQUIRE(!group_open() || (dtype == SPA_BF16 && Dh == 32 && at_tokens), SPA_ERR_UNSUPPORTED,
              "%s: this form cannot be part of a group", fn);
  if (dtype == SPA_F32) {
    const dim3 grid((max_seqlen + 127) / 128, H, B), block(128);
#define SPA_BWD_F32(D)                                                                                        \
  hipLaunchKernelGGL((attn_bwd_f32_kernel<D, false>), grid, block, 0, st, (const float*)q, (const float*)k,   \
                     (const float*)v, (long)q_row_stride, (long)k_row_stride, (long)v_row_stride,             \
                     (const float*)out, (const float*)dout, lse, dvec, ls, cu_seqlens, H, scale, (float*)dq,  \
                     (long)dq_row_stride, (float*)nullptr, 0L, tok);                                          \
  hipLaunchKernelGGL((attn_bwd_f32_kernel<D, true>), grid, block, 0, st, (const float*)q, (const float*)k,    \
                     (const float*)v, (long)q_row_stride, (long)k_row_stride, (long)v_row_stride,             \
                     (const float*)out, (const float*)dout, lse, dvec, ls, cu_seqlens, H, scale, (float*)dk,  \
                     (long)dk_row_stride, (float*)dv, (long)dv_row_stride, tok)
    if (Dh == 32) { SPA_BWD_F32(32); } else { SPA_BWD_F32(64); }
#undef SPA_BWD_F32
  } else {
    const BwdArgs args = {(const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (long)q_row_stride, (long)k_row_stride,
                          (long)v_row_stride, v_scores, (const __bf16*)out, (const __bf16*)dout, lse, ls, cu_seqlens, H, B,
                          scale, (__bf16*)dq, (__bf16*)dk, (__bf16*)dv, (long)dq_row_stride, (long)dk_row_stride,
                          (long)dv_row_stride, tok, dvec, (max_seqlen + kBwdRows - 1) / kBwdRows};
    if (one_kernel) {
      const int nw = (max_seqlen + 31) / 32;
      SPA_REQUIRE((long)B * H < 2147483647L, SPA_ERR_INVALID_ARG, "%s: B*H must be < 2^31", fn);
#define SPA_BWD_SHORT(D, G)                                                                                     \
  do {                                                                                                          \
    const size_t smem = bwd_short_lds_bytes<D>(nw);                                                             \
    const hipError_t attr = hipFuncSetAttribute((const void*)attn_bwd_short_bf16_kernel<D, G>,                  \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);         \
    SPA_REQUIRE(attr == hipSuccess, SPA_ERR_HIP, "%s: cannot reserve %zu bytes of LDS", fn, smem);              \
    hipLaunchKernelGGL((attn_bwd_short_bf16_kernel<D, G>), dim3((unsigned)(B * H)), dim3(64 * nw), smem, st, args); \
  } while (0)
      if (v_scores != nullptr) {
        if (Dh == 32) SPA_BWD_SHORT(32, true); else SPA_BWD_SHORT(64, true);
      } else {
        if (Dh == 32) SPA_BWD_SHORT(32, false); else SPA_BWD_SHORT(64, false);
      }
#undef SPA_BWD_SHORT
      return check_launch(fn);
    }
    // long segments: D first, then both roles in one launch
    const int nblk = args.nblk;
    SPA_REQUIRE(2 * ((long)H * B + 8) * nblk < 2147483647L, SPA_ERR_INVALID_ARG, "%s: B*H*blocks must be < 2^30", fn);
    const bool resident = nblk <= 4 && live_tiles_apply(H, B);
    const unsigned all = 2 * xcd_grid(nblk, H, B), grid = resident && !group_open() ? std::min(all, (unsigned)bwd_long_slots(Dh)) : all;
    const unsigned dgrid = dvec_blocks((long)B * max_seqlen, H, Dh);
    if (group_open()) {
      if (!have_d)
        if (int rc = g_noted_dvec[v_scores != nullptr].add(fn, args, dgrid)) return rc;
      return g_noted[v_scores != nullptr].add(fn, args, grid);
    }
#define SPA_BWD_MODE(KERNEL, D)                                                                                 \
  do {                                                                                                          \
    if (v_scores != nullptr) hipLaunchKernelGGL((KERNEL<D, kGated>), dim3(grid), dim3(kBwdThreads), 0, st, args); \
    else if (at_tokens) hipLaunchKernelGGL((KERNEL<D, kTokens>), dim3(grid), dim3(kBwdThreads), 0, st, args);   \
    else hipLaunchKernelGGL((KERNEL<D, kPacked>), dim3(grid), dim3(kBwdThreads), 0, st, args);                  \
  } while (0)
#define SPA_BWD_LONG(D)                                                                                         \
  do {                                                                                                          \
    if (!have_d) hipLaunchKernelGGL((attn_bwd_dvec_kernel<D>), dim3(dgrid), dim3(256), 0, st, args);            \
    if (resident) SPA_BWD_MODE(attn_bwd_resident_bf16_kernel, D);                                               \
    else SPA_BWD_MODE(attn_bwd_long_bf16_kernel, D);                                                            \
  } while (0)
    if (Dh == 32) SPA_BWD_LONG(32); else SPA_BWD_LONG(64);
#undef SPA_BWD_LONG
#undef SPA_BWD_MODE
  }
  return check_launch(fn);
}

extern "C" int spa_packed_attention_bwd(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                        int64_t k_row_stride, int64_t v_row_stride, const void* out,
                                        const void* dout, const float* lse, const int32_t* cu_seqlens, int B,
                                        int max_seqlen, int H, int Dh, int dtype, float softmax_scale,
                                        void* dq, void* dk, void* dv, int64_t dq_row_stride,
                                        int64_t dk_row_stride, int64_t dv_row_stride, void* workspace,
                                        size_t workspace_bytes, void* stream) {
  return attention_bwd_common("spa_packed_attention_bwd", q, k, v, q_row_stride, k_row_stride, v_row_stride, out,
                              dout, lse, cu_seqlens, B, max_seqlen, H, Dh, dtype, softmax_scale, dq, dk, dv,
                              dq_row_stride, dk_row_stride, dv_row_stride, workspace, workspace_bytes,
                              TokenIO{nullptr, nullptr, 0}, stream, false);
}

extern "C" int spa_packed_attention_bwd_spread(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                               int64_t k_row_stride, int64_t v_row_stride, const void* out,
                                               const void* dout, const float* lse, const int32_t* cu_seqlens, int B,
                                               int max_seqlen, int H, int Dh, int dtype, float softmax_scale,
                                               void* dq, void* dk, void* dv, int64_t dq_row_stride,
                                               int64_t dk_row_stride, int64_t dv_row_stride, void* workspace,
                                               size_t workspace_bytes, void* stream) {
  return attention_bwd_common("spa_packed_attention_bwd_spread", q, k, v, q_row_stride, k_row_stride, v_row_stride, out,
                              dout, lse, cu_seqlens, B, max_seqlen, H, Dh, dtype, softmax_scale, dq, dk, dv,
                              dq_row_stride, dk_row_stride, dv_row_stride, workspace, workspace_bytes,
                              TokenIO{nullptr, nullptr, 0}, stream, true);
}

extern "C" int spa_packed_attention_bwd_tokens(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                               int64_t k_row_stride, int64_t v_row_stride, const void* out,
                                               const void* dy, const float* lse, const int32_t* cu_seqlens, int B,
                                               int max_seqlen, int H, int Dh, int dtype, float softmax_scale,
                                               const int32_t* gather_idx, const int32_t* inv_pos, int64_t rows,
                                               void* dq, void* dk, void* dv, int64_t dq_row_stride,
                                               int64_t dk_row_stride, int64_t dv_row_stride, void* workspace,
                                               size_t workspace_bytes, void* stream) {
  const char* fn = "spa_packed_attention_bwd_tokens";
  SPA_REQUIRE(gather_idx && inv_pos, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(rows >= 1 && rows < 2147483647L, SPA_ERR_INVALID_ARG, "%s: rows must be in [1, 2^31)", fn);
  return attention_bwd_common(fn, q, k, v, q_row_stride, k_row_stride, v_row_stride, out, dy, lse, cu_seqlens, B,
                              max_seqlen, H, Dh, dtype, softmax_scale, dq, dk, dv, dq_row_stride, dk_row_stride,
                              dv_row_stride, workspace, workspace_bytes, TokenIO{gather_idx, inv_pos, (long)rows},
                              stream, false);
}

extern "C" int spa_gated_attention_bwd_tokens(const void* q, const void* k, const void* x, int64_t q_row_stride,
                                              int64_t k_row_stride, int64_t x_row_stride, const float* scores,
                                              const void* out, const void* dy, const float* lse, const int32_t* cu_seqlens,
                                              int B, int max_seqlen, int H, int Dh, int dtype, float softmax_scale,
                                              const int32_t* gather_idx, const int32_t* inv_pos, int64_t rows, void* dq,
                                              void* dk, void* d_rg, int64_t dq_row_stride, int64_t dk_row_stride,
                                              int64_t d_rg_row_stride, void* workspace, size_t workspace_bytes, void* stream) {
  const char* fn = "spa_gated_attention_bwd_tokens";
  SPA_REQUIRE(scores && gather_idx && inv_pos, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(rows >= 1 && rows < 2147483647L, SPA_ERR_INVALID_ARG, "%s: rows must be in [1, 2^31)", fn);
  SPA_REQUIRE(dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: bf16 only (use spa_pack_pair + spa_packed_attention_bwd_tokens)", fn);
  return attention_bwd_common(fn, q, k, x, q_row_stride, k_row_stride, x_row_stride, out, dy, lse, cu_seqlens, B,
                              max_seqlen, H, Dh, dtype, softmax_scale, dq, dk, d_rg, dq_row_stride, dk_row_stride,
                              d_rg_row_stride, workspace, workspace_bytes, TokenIO{gather_idx, inv_pos, (long)rows},
                              stream, false, scores);
}

extern "C" int spa_gated_attention_bwd_tokens_spread(const void* q, const void* k, const void* x, int64_t q_row_stride,
                                                     int64_t k_row_stride, int64_t x_row_stride, const float* scores,
                                                     const void* out, const void* dy, const float* lse, const int32_t* cu_seqlens,
                                                     int B, int max_seqlen, int H, int Dh, int dtype, float softmax_scale,
                                                     const int32_t* gather_idx, const int32_t* inv_pos, int64_t rows, void* dq,
                                                     void* dk, void* d_rg, int64_t dq_row_stride, int64_t dk_row_stride,
                                                     int64_t d_rg_row_stride, void* workspace, size_t workspace_bytes, void* stream) {
  const char* fn = "spa_gated_attention_bwd_tokens_spread";
  SPA_REQUIRE(scores && gather_idx && inv_pos, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(rows >= 1 && rows < 2147483647L, SPA_ERR_INVALID_ARG, "%s: rows must be in [1, 2^31)", fn);
  SPA_REQUIRE(dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: bf16 only (use spa_pack_pair + spa_packed_attention_bwd_tokens)", fn);
  return attention_bwd_common(fn, q, k, x, q_row_stride, k_row_stride, x_row_stride, out, dy, lse, cu_seqlens, B,
                              max_seqlen, H, Dh, dtype, softmax_scale, dq, dk, d_rg, dq_row_stride, dk_row_stride,
                              d_rg_row_stride, workspace, workspace_bytes, TokenIO{gather_idx, inv_pos, (long)rows},
                              stream, true, scores);
}

extern "C" int spa_gated_attention_bwd_tokens_dvec(const void* q, const void* k, const void* x, int64_t q_row_stride,
                                                   int64_t k_row_stride, int64_t x_row_stride, const float* scores,
                                                   const void* out, const void* dy, const float* lse, const int32_t* cu_seqlens,
                                                   int B, int max_seqlen, int H, int Dh, int dtype, float softmax_scale,
                                                   const int32_t* gather_idx, const int32_t* inv_pos, int64_t rows, void* dq,
                                                   void* dk, void* d_rg, int64_t dq_row_stride, int64_t dk_row_stride,
                                                   int64_t d_rg_row_stride, void* workspace, size_t workspace_bytes,
                                                   const void* y, void* stream) {
  const char* fn = "spa_gated_attention_bwd_tokens_dvec";
  SPA_REQUIRE(scores && gather_idx && inv_pos && y, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(rows >= 1 && rows < 2147483647L, SPA_ERR_INVALID_ARG, "%s: rows must be in [1, 2^31)", fn);
  SPA_REQUIRE(dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: bf16 only (use spa_pack_pair + spa_packed_attention_bwd_tokens)", fn);
  return attention_bwd_common(fn, q, k, x, q_row_stride, k_row_stride, x_row_stride, out, dy, lse, cu_seqlens, B,
                              max_seqlen, H, Dh, dtype, softmax_scale, dq, dk, d_rg, dq_row_stride, dk_row_stride,
                              d_rg_row_stride, workspace, workspace_bytes, TokenIO{gather_idx, inv_pos, (long)rows},
                              stream, true, scores, true);
}
