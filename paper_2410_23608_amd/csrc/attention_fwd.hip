// Masked multi-head self-attention on packed tokens (Section 3.2, last paragraph): a token
// attends only to tokens of its own image.  The mask is never built: a workgroup works on
// one (image, head, query block) and walks the keys of that image's segment only.
//
// bf16 path (MFMA, fp32 softmax).  One wave owns 32 queries.  It computes the TRANSPOSED
// score tile S^T = K Q^T with v_mfma_f32_32x32x16_bf16, so that in the accumulator layout
// (column = lane % 32, 16 rows per lane) a lane holds 16 keys of ONE query: row max and
// row sum are in-lane reductions plus one exchange with lane ^ 32, the running max / sum /
// rescale factor are one scalar per lane, and the bf16-rounded probabilities are already
// in the B-operand layout of the second product O^T = V^T P^T — no trip through LDS.
// K tiles sit in LDS row-major (A operand: 16-byte reads), V tiles are stored transposed.
//
// fp32 path (small fp32 workload): the same transposed tiles on the fp32 MFMA, in registers only.
#include <cmath>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <type_traits>

#include "attn_tiles.h"
#include "group.h"
#include "spa_common.h"

namespace spa {

// Optional fused scatter-back (the unpack step folded into the attention kernel): packed
// output row j goes to y[gather_idx[j]] (plus base), and every workgroup first fills its
// share of the rows that bypass attention (inv_pos < 0) with base or zero.  All-null = off.
// y is the path's final output: nothing here reads it again, so its stores are non-temporal
// (they do not push the packed rows the next launches read out of the caches).
struct Scatter {
  const int32_t* gather_idx;   // [B*N] packed row -> flat token
  const int32_t* inv_pos;      // [B*N] flat token -> packed row or -1
  const void* base;            // [B*N, C] residual or nullptr
  void* y;                     // [B*N, C]
  int N;                       // tokens per image; in flat mode all rows of y (B*N)
  int flat;                    // 0: segment s fills the bypassing rows of image s (segments are images)
                               // 1: segments are not images (containers): the rows of y are dealt
                               //    evenly to all (segment, part) work units
  int gathered;                // 1: q, k, v are NOT packed: the row of packed position j is row
                               //    gather_idx[j] of q, k, v (token positions); packing then only
                               //    builds the index and no row is copied before the attention
  const uint8_t* mask;         // [B*N] or nullptr: when given, a token bypasses attention iff its mask byte is 0
                               //    (used in place of inv_pos by the form that is given no packing index)
  const __bf16* dy = nullptr;  // kFwdGatedD: the gradient of y, where it is there already, and
  float* dvec = nullptr;       //    D_i = <dy_i, out_i> of every (head, packed row), laid out as lse, for the backward
};
__device__ __forceinline__ bool bypasses(const Scatter& sc, long row) {
  return sc.mask != nullptr ? sc.mask[row] == 0 : sc.inv_pos[row] < 0;
}

// Operands and results of the bf16 kernels that can share a launch.
struct FwdArgs {
  const __bf16 *q, *k, *v;
  long qs, ks, vs;
  const float* v_scores;       // kFwdGated: score of every token
  const int32_t *cu, *key_lens;
  int n_pad, H;
  float scale_log2;
  __bf16* out;
  float* lse;
  long lse_stride;
  Scatter sc;
  int B, nqb, ntile;
  int waves;                   // launch groups: waves a unit of the short form (1 or 2)
};

// Row of q / k / v that holds packed position j of a segment starting at packed row row0:
// gi = gather_idx + row0 when the rows are gathered through the index, else null.
// GATHER is a compile-time property of every bf16 kernel: with packed rows (kFwdPacked) the index is known to be
// absent and the row addresses stay affine in the loop counters (pointer increments), with gathered
// rows every row address is a multiply on a loaded index.  kFwdGated: gathered, and a v row is multiplied by
// Sigmoid(score of its token) and rounded to bf16 on its way to LDS, as a packed r_g holds it.
// kFwdGatedD: and D of the backward (Scatter::dvec).
constexpr int kFwdPacked = 0, kFwdGathered = 1, kFwdGated = 2, kFwdGatedD = 3, kFwdForms = 4;
constexpr bool is_gated(int gather) { return gather >= kFwdGated; }
template <int GATHER>
__device__ __forceinline__ const int32_t* gather_base(const Scatter& sc, long row0) {
  return GATHER ? sc.gather_idx + row0 : nullptr;
}
__device__ __forceinline__ long source_row(const int32_t* gi, long row0, int j) {
  return gi != nullptr ? (long)gi[j] : row0 + j;
}
// Element offset of a gathered row: one 32 x 32 -> 64 bit multiply (the host checks that rows and
// strides are below 2^31).
__device__ __forceinline__ long row_offset(int row, long stride) {
  return (long)((unsigned long)(uint32_t)row * (uint32_t)stride);
}

// The rows whose bypass fill falls to work unit (segment `seg` of `nseg`, part `part` of `nparts`):
// tokens [t0, t1) of image b (flat mode: b = 0 and the range is over all rows of y).
struct FillRange {
  int b, t0, t1;
};
__device__ __forceinline__ FillRange fill_range(const Scatter& sc, int seg, int nseg, int part, int nparts) {
  FillRange f = {0, 0, 0};
  if (sc.y == nullptr) return f;
  if (!sc.flat) {
    const int per = (sc.N + nparts - 1) / nparts;
    f.b = seg;
    f.t0 = min(sc.N, part * per);
    f.t1 = min(sc.N, (part + 1) * per);
  } else {
    const long units = (long)nseg * nparts, u = (long)seg * nparts + part;
    const long per = (sc.N + units - 1) / units;
    f.t0 = (int)min((long)sc.N, u * per);
    f.t1 = (int)min((long)sc.N, (u + 1) * per);
  }
  return f;
}

// Fill the head slice [h*DH, (h+1)*DH) of the bypassing rows among tokens [t0, t1) of image b.
// Shared by `nthreads` threads, this one being number `tid` of them.
template <typename T, int DH>
__device__ __forceinline__ void scatter_fill(const Scatter& sc, int b, int t0, int t1, int h, long C, int tid,
                                             int nthreads) {
  constexpr int VE = 16 / sizeof(T), CPR = DH / VE;
  const long tok0 = (long)b * sc.N;
  const int work = (t1 - t0) * CPR;
  for (int i = tid; i < work; i += nthreads) {
    const int t = t0 + i / CPR, c = i % CPR;
    if (bypasses(sc, tok0 + t)) {
      const long off = (tok0 + t) * C + h * DH + c * VE;
      uintx4 val = {0u, 0u, 0u, 0u};
      if (sc.base != nullptr) val = *reinterpret_cast<const uintx4*>(static_cast<const T*>(sc.base) + off);
      __builtin_nontemporal_store(val, reinterpret_cast<uintx4*>(static_cast<T*>(sc.y) + off));
    }
  }
}

// One wave fills the bypassing rows among rows [r0, r1) of y: the lanes test 64 rows at a time and list those
// that need it, then the wave goes over their 16-byte chunks, all lanes at work whatever the row length, four
// steps of loads in flight.
template <typename T>
__device__ __forceinline__ void scatter_fill_rows(const Scatter& sc, long r0, long r1, long C, int lane) {
  constexpr int VE = 16 / sizeof(T), U = 4;
  const int cpr = (int)(C / VE), dr = kWave / cpr, dc = kWave % cpr;
  for (long rb = r0; rb < r1; rb += kWave) {
    const long row = rb + lane;
    const bool mine = row < r1 && bypasses(sc, row);
    const uint64_t m = __ballot(mine);
    const int n = __popcll(m), below = lanes_below(m);
    const int list = __builtin_amdgcn_ds_permute((mine ? below : n + lane - below) << 2, lane);   // lane i: i-th such row
    int r = lane / cpr, c = lane % cpr;
    for (int left = n * cpr; left > 0; left -= U * kWave) {
      uintx4 val[U];
      T* dst[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        ok[u] = r < n;
        const long off = (rb + __builtin_amdgcn_ds_bpermute((r & 63) << 2, list)) * C + c * VE;
        dst[u] = static_cast<T*>(sc.y) + off;
        val[u] = uintx4{0u, 0u, 0u, 0u};
        if (sc.base != nullptr && ok[u]) val[u] = *reinterpret_cast<const uintx4*>(static_cast<const T*>(sc.base) + off);
        r += dr;
        c += dc;
        if (c >= cpr) {
          c -= cpr;
          ++r;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (ok[u]) __builtin_nontemporal_store(val[u], reinterpret_cast<uintx4*>(dst[u]));
    }
  }
}

// ------------------------------------------------------------------------- bf16 / MFMA
// The running maximum before any score: the lowest finite number, so that keys whose scores are all -inf (products that
// overflow; a wave of a split unit may see no others) weigh exp(-inf - m) = 0 instead of exp(-inf + inf) = NaN.
constexpr float kNoScore = -std::numeric_limits<float>::max();
// Per-wave state of the softmax: O^T accumulators (rows = head dim, cols = this wave's 32
// queries), running maximum m of the scores (log2 domain, scale folded in; see fwd_exp) and running
// sum l (the two halves of the wave keep partial sums that are added at the end).
template <int DH>
struct FwdAcc {
  floatx16 o[DH / 32];
  float m, l;
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int d = 0; d < DH / 32; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
    m = kNoScore;
    l = 0.f;
  }
};

// When a group's fragments are read from LDS.  kReadLate: each where a product needs it.  kReadSome: K before the first score
// product, the first of V before the softmax, the others right after it.  kReadAll: all of V before the softmax, which
// covers the reads.
enum FragReads { kReadLate, kReadSome, kReadAll };

// Score sub-tiles of one group of GSB*32 keys: S^T = K Q^T (rows = keys, cols = queries).
// key0 = first key of the group inside the LDS tile, rem = valid keys of the tile.
// EARLY: all of its K fragments are read before the first product.
template <int DH, int RS, int GSB, bool FULL, bool EARLY = false>
__device__ __forceinline__ void fwd_scores(const __bf16* kbuf, int key0, int rem, const bf16x8 (&qf)[DH / 16],
                                           floatx16 (&s)[GSB], int l32, int hh) {
  auto k_frag = [&](int sb, int kk) {
    return *reinterpret_cast<const bf16x8*>(&kbuf[(key0 + sb * 32 + l32) * RS + kk * 16 + hh * 8]);
  };
  bf16x8 kf[EARLY ? GSB : 1][DH / 16];
  if constexpr (EARLY) {
#pragma unroll
    for (int sb = 0; sb < GSB; ++sb)
#pragma unroll
      for (int kk = 0; kk < DH / 16; ++kk) kf[sb][kk] = k_frag(sb, kk);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int sb = 0; sb < GSB; ++sb) {
    const int k0 = key0 + sb * 32;
    if (FULL || EARLY || k0 < rem) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[sb][r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < DH / 16; ++kk)
        s[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(EARLY ? kf[EARLY ? sb : 0][kk] : k_frag(sb, kk), qf[kk], s[sb], 0, 0, 0);
      if (!FULL && rem - k0 < 32) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (k0 + acc_row(r, hh) >= rem) s[sb][r] = -INFINITY;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[sb][r] = -INFINITY;
    }
  }
}

// The online softmax of a group of GSB*32 keys: P = exp2(S scale - m) with m the running maximum of the row, O and
// l rescaled where it moved.  The maximum is what keeps the results accurate, not only in range: the largest
// probability of a row is then exactly 1 and rounds to bf16 without an error, so that a row whose weight lies on one
// key returns that key's V row and dP - D cancels there in the backward.  Against any other reference it is rounded by
// up to 2^-9 while l adds the unrounded values: the error of the output against 64 bits grows by 1.1, 1.25 and 1.35
// for normal q and k of sigma 1, 1.5 and 2, that of dq and dk by up to 1.5.  A fixed reference with a rescue by the
// maximum was faster (us a step: 8 images of 4200 tokens, 5-40 %, 8 heads of 32, 35.5 against 38.7; 64 x 196 tokens,
// 6 heads of 64, 15.7 against 16.8) and not kept for that loss.
template <int DH, int GSB, bool FULL>
__device__ __forceinline__ void fwd_exp(const floatx16 (&s)[GSB], int key0, int rem, FwdAcc<DH>& acc, float scale_log2,
                                        bf16x8 (&pb)[GSB][2]) {
  // (maximum, not fmaxf: a NaN stays one, so that no operand is canonicalised first, 6 instructions fewer of 145 a tile of 64
  // keys; us a step, 32 x 4200 tokens, 5-40 %, 8 heads of 32, 85.0 -> 84.4, 8 images 32.2 -> 31.7, 64 x 196 tokens, 6 heads
  // of 64, 15.2 -> 15.1.  A row with a NaN among its scores is NaN either way.)
  float mx = s[0][0];
#pragma unroll
  for (int sb = 0; sb < GSB; ++sb)
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = __builtin_elementwise_maximum(mx, s[sb][r]);
  const float m_new = __builtin_elementwise_maximum(acc.m, max_across_halves(mx) * scale_log2);
  if (__ballot(m_new != acc.m) != 0) {                 // some query's running max moved: rescale
    const float alpha = __builtin_amdgcn_exp2f(acc.m - m_new);
    acc.l *= alpha;
#pragma unroll
    for (int d = 0; d < DH / 32; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc.o[d][r] *= alpha;
    acc.m = m_new;
  }
  float psum = 0.f;
#pragma unroll
  for (int sb = 0; sb < GSB; ++sb)
    if (FULL || key0 + sb * 32 < rem) {
      float p[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        p[r] = __builtin_amdgcn_exp2f(fmaf(s[sb][r], scale_log2, -m_new));
        psum += p[r];
      }
#pragma unroll
      for (int mf = 0; mf < 2; ++mf) {
        floatx8 pf;
#pragma unroll
        for (int j = 0; j < 8; ++j) pf[j] = p[8 * mf + j];
        pb[sb][mf] = float_to_bf16x8(pf);
      }
    }
  acc.l += psum;
}

// The probabilities of a group of GSB*32 keys, then O^T += V^T P^T.  V^T at vbuf (row stride TS), the
// group's keys at column vcol; TS == 0: V rows as they lie in memory (row stride DH + 8, the group's keys
// from row vcol), the V^T fragments then come from the transposing LDS read.
// READS: when its V^T fragments are read.
template <int DH, int TS, int GSB, bool FULL, int READS = kReadLate>
__device__ __forceinline__ void fwd_softmax_pv(const floatx16 (&s)[GSB], const __bf16* vbuf, int vcol, int key0, int rem,
                                               FwdAcc<DH>& acc, float scale_log2, int l32, int hh) {
  constexpr int DB = DH / 32;
  auto v_frag = [&](int sb, int mf, int d) {
    return TS == 0 ? transposed_frag_rowmajor<DH + 8>(vbuf, d, vcol + sb * 32, mf, l32 + 32 * hh)
                   : transposed_frag<TS == 0 ? 1 : TS>(vbuf, d * 32 + l32, vcol + sb * 32, mf, hh);
  };
  constexpr int F = 2 * GSB, BEFORE = READS == kReadAll ? F : READS == kReadSome ? 1 : 0;    // (of each 32 columns)
  bf16x8 vf[READS != kReadLate ? GSB : 1][2][DB], pb[GSB][2];
  auto read = [&](int from, int to) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int d = 0; d < DB; ++d)
        if (f >= from && f < to) vf[READS != kReadLate ? f >> 1 : 0][f & 1][d] = v_frag(f >> 1, f & 1, d);
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (BEFORE > 0) read(0, BEFORE);
  fwd_exp<DH, GSB, FULL>(s, key0, rem, acc, scale_log2, pb);
  if constexpr (READS == kReadSome) read(BEFORE, F);
#pragma unroll
  for (int sb = 0; sb < GSB; ++sb)
    if (FULL || key0 + sb * 32 < rem) {
#pragma unroll
      for (int mf = 0; mf < 2; ++mf)
#pragma unroll
        for (int d = 0; d < DB; ++d) {
          const bf16x8 a = READS != kReadLate ? vf[READS != kReadLate ? sb : 0][mf][d] : v_frag(sb, mf, d);
          acc.o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[sb][mf], acc.o[d], 0, 0, 0);
        }
    }
}

// One tile of NSB*32 keys held in LDS (K rows at kbuf, row stride RS; V^T at vbuf, row
// stride TS, the tile's keys starting at column vcol0), processed in groups of 64 keys with
// a two-stage software pipeline: the score MFMAs of group g+1 are issued before the softmax
// VALU work of group g, and that group's P V MFMAs run under the next group's softmax, so
// the matrix pipe and the vector ALU overlap inside one wave.  rem = valid keys in the tile;
// FULL = every key valid (no masking code).
template <int DH, int RS, int TS, int NSB, bool FULL>
__device__ __forceinline__ void fwd_process_tile(const __bf16* kbuf, const __bf16* vbuf, int vcol0, int rem,
                                                 const bf16x8 (&qf)[DH / 16], FwdAcc<DH>& acc,
                                                 float scale_log2, int l32, int hh) {
  constexpr int GSB = NSB >= 4 ? 2 : 1;     // sub-tiles per softmax group
  constexpr int NG = NSB / GSB;
  floatx16 s[2][GSB];
  fwd_scores<DH, RS, GSB, FULL>(kbuf, 0, rem, qf, s[0], l32, hh);
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int key0 = g * GSB * 32;
    if (!FULL && key0 >= rem) break;
    if (g + 1 < NG && (FULL || key0 + GSB * 32 < rem))
      fwd_scores<DH, RS, GSB, FULL>(kbuf, key0 + GSB * 32, rem, qf, s[(g + 1) & 1], l32, hh);
    fwd_softmax_pv<DH, TS, GSB, FULL>(s[g & 1], vbuf, vcol0 + key0, key0, rem, acc, scale_log2, l32, hh);
  }
}

// Output stage, phase 1: normalise this wave's O^T accumulators and park the 32 x DH bf16
// tile in LDS (row = query, row stride RS), so that phase 2 can write whole rows.
// Also writes lse.  Called by every lane of a live wave.
template <int DH, int RS>
__device__ __forceinline__ void fwd_park(FwdAcc<DH>& acc, bool q_ok, bool have_keys, __bf16* tile,
                                         float* lse_ptr, int l32, int hh) {
  const float l_tot = sum_across_halves(acc.l);
  const float inv = have_keys ? 1.0f / l_tot : 0.f;
#pragma unroll
  for (int d = 0; d < DH / 32; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      floatx4 f = {acc.o[d][4 * g] * inv, acc.o[d][4 * g + 1] * inv, acc.o[d][4 * g + 2] * inv,
                   acc.o[d][4 * g + 3] * inv};
      *reinterpret_cast<bf16x4*>(&tile[l32 * RS + d * 32 + 8 * g + 4 * hh]) = __builtin_convertvector(f, bf16x4);
    }
  if (q_ok && lse_ptr != nullptr && hh == 0)
    *lse_ptr = have_keys ? (acc.m + __log2f(l_tot)) * 0.69314718055994531f : -INFINITY;
}

// Output stage, phase 2 (after a barrier): the wave copies its parked tile to global memory,
// consecutive lanes writing consecutive 16-byte chunks of a row.  nrows = valid rows (<= 32);
// prow0 = packed row of the tile's first row, y_row = row of y of lane % 32's row.  out may be null when only y is wanted.
// D (dvec): also the products of the rows with those of sc.dy, to dvec[packed row].
template <int DH, int RS, bool D = false>
__device__ __forceinline__ void fwd_flush(const __bf16* tile, __bf16* out, const Scatter& sc, int y_row, long prow0, int h,
                                          long C, int nrows, int lane, float* dvec = nullptr) {
  constexpr int CPR = DH / 8;
  if constexpr (D) {
    constexpr int PASSES = 32 * CPR / 64;
    bf16x8 g[PASSES];
#pragma unroll
    for (int t = 0; t < PASSES; ++t) {
      const int i = lane + 64 * t, r = i / CPR, token = __builtin_amdgcn_ds_bpermute(r << 2, y_row);
      g[t] = zero_bf16x8();
      if (r < nrows) g[t] = *reinterpret_cast<const bf16x8*>(sc.dy + (long)token * C + h * DH + i % CPR * 8);
    }
#pragma unroll
    for (int t = 0; t < PASSES; ++t) {
      const int i = lane + 64 * t, r = i / CPR;
      const floatx8 of = bf16x8_to_float(*reinterpret_cast<const bf16x8*>(&tile[r * RS + i % CPR * 8]));
      const floatx8 gf = bf16x8_to_float(g[t]);
      float d = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) d = fmaf(of[e], gf[e], d);
      d = adjacent_sum<CPR>(d);
      if (r < nrows && i % CPR == 0) dvec[prow0 + r] = d;
    }
  }
#pragma unroll
  for (int i = lane; i < 32 * CPR; i += 64) {
    const int r = i / CPR, c = i % CPR, token = __builtin_amdgcn_ds_bpermute(r << 2, y_row);
    if (r < nrows) {
      bf16x8 val = *reinterpret_cast<const bf16x8*>(&tile[r * RS + c * 8]);
      if (out != nullptr) *reinterpret_cast<bf16x8*>(out + (prow0 + r) * C + h * DH + c * 8) = val;
      if (sc.y != nullptr) {
        const long off = (long)token * C + h * DH + c * 8;
        if (sc.base != nullptr) {
          const floatx8 bv = bf16x8_to_float(*reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(sc.base) + off));
          val = float_to_bf16x8(bf16x8_to_float(val) + bv);
        }
        __builtin_nontemporal_store(val, reinterpret_cast<bf16x8*>(static_cast<__bf16*>(sc.y) + off));
      }
    }
  }
}

// Register staging of key/value rows on their way to LDS: task i = 16-byte chunk column
// c = i % CPR of the row pair (2*(i / CPR), +1); K goes row-major, V transposed.
template <int DH, int THREADS, int TASKS, int GATHER>
struct KvStage {
  static constexpr int CPR = DH / 8;
  static constexpr int TPT = (TASKS + THREADS - 1) / THREADS;
  static constexpr int RPP = 2 * THREADS / CPR;   // rows one pass of the workgroup covers
  static_assert(THREADS % CPR == 0, "a thread keeps its chunk column over the passes");
  bf16x8 kreg[TPT][2], vreg[TPT][2];

  // The rows the next load() fetches: keys [kt_, kt_ + tile) of a segment of nk_ keys whose packed rows
  // start at row0_.  Packed rows need no per-lane address arithmetic: the address is a uniform base
  // (segment, tile, pass) plus a 32-bit per-lane offset that never changes.  Gathered rows have their
  // token rows loaded here, one tile ahead of load(), so the row loads never wait for an index.
  int tok_rows[TPT][2];
  long row0_;
  int kt_, nk_;

  __device__ __forceinline__ bool valid(int t, int u) const {
    const int i = threadIdx.x + t * THREADS;
    return i < TASKS && kt_ + 2 * (i / CPR) + u < nk_;
  }
  __device__ __forceinline__ void index(const int32_t* gi, long row0, int kt, int nk) {
    row0_ = row0;
    kt_ = kt;
    nk_ = nk;
    if (GATHER) {
      if (TASKS % THREADS == 0 && kt + 2 * TASKS / CPR <= nk) {      // a whole tile: no predicates
#pragma unroll
        for (int t = 0; t < TPT; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u) tok_rows[t][u] = gi[kt + 2 * ((threadIdx.x + t * THREADS) / CPR) + u];
      } else {
#pragma unroll
        for (int t = 0; t < TPT; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (valid(t, u)) tok_rows[t][u] = gi[kt + 2 * ((threadIdx.x + t * THREADS) / CPR) + u];
      }
    }
  }
  // The row loads; rows past the segment read as zero
  __device__ __forceinline__ void load(const __bf16* kh, const __bf16* vh, long ks, long vs) {
    const int c = threadIdx.x % CPR, lrow = 2 * (threadIdx.x / CPR);
    const uint32_t koff = (uint32_t)lrow * (uint32_t)ks + c * 8, voff = (uint32_t)lrow * (uint32_t)vs + c * 8;
    // a tile that lies wholly inside the segment (all but the last one): no predicates, no zero fill
    if (TASKS % THREADS == 0 && kt_ + 2 * TASKS / CPR <= nk_) {
#pragma unroll
      for (int t = 0; t < TPT; ++t) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const __bf16 *kp, *vp;
          if (GATHER) {
            kp = kh + row_offset(tok_rows[t][u], ks) + c * 8;
            vp = vh + row_offset(tok_rows[t][u], vs) + c * 8;
          } else {
            const long r = row0_ + kt_ + t * RPP + u;     // uniform
            kp = kh + r * ks + koff;
            vp = vh + r * vs + voff;
          }
          kreg[t][u] = *reinterpret_cast<const bf16x8*>(kp);
          vreg[t][u] = *reinterpret_cast<const bf16x8*>(vp);
        }
      }
      return;
    }
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        kreg[t][u] = zero_bf16x8();
        vreg[t][u] = zero_bf16x8();
        if (valid(t, u)) {
          const __bf16 *kp, *vp;
          if (GATHER) {
            kp = kh + row_offset(tok_rows[t][u], ks) + c * 8;
            vp = vh + row_offset(tok_rows[t][u], vs) + c * 8;
          } else {
            const long r = row0_ + kt_ + t * RPP + u;     // uniform
            kp = kh + r * ks + koff;
            vp = vh + r * vs + voff;
          }
          kreg[t][u] = *reinterpret_cast<const bf16x8*>(kp);
          vreg[t][u] = *reinterpret_cast<const bf16x8*>(vp);
        }
      }
    }
  }
  // K rows -> kbuf[row * RS], V -> vbuf[d * TS + col0 + row]
  template <int RS, int TS>
  __device__ __forceinline__ void store(__bf16* kbuf, __bf16* vbuf, int col0) const {
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
      const int i = threadIdx.x + t * THREADS;
      if (i < TASKS) {
        const int c = i % CPR, r0 = 2 * (i / CPR);
        *reinterpret_cast<bf16x8*>(&kbuf[r0 * RS + c * 8]) = kreg[t][0];
        *reinterpret_cast<bf16x8*>(&kbuf[(r0 + 1) * RS + c * 8]) = kreg[t][1];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          bf16x2 pr = {vreg[t][0][e], vreg[t][1][e]};
          *reinterpret_cast<bf16x2*>(&vbuf[(c * 8 + e) * TS + col0 + r0]) = pr;
        }
      }
    }
  }
};

template <int DH>
__device__ __forceinline__ void load_q_frags(const __bf16* qrow, bool q_ok, int hh, bf16x8 (&qf)[DH / 16]) {
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk) {
    qf[kk] = zero_bf16x8();
    if (q_ok) qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + kk * 16 + hh * 8);
  }
}

// Long segments.  Workgroup = NW waves x 32 queries; the keys of the segment stream through LDS in tiles of BN,
// double-buffered: while a tile is consumed the next one is in flight from global memory into registers
// (PairStage), and is written to the other LDS buffer before the single barrier that ends the iteration.  K and V
// lie in LDS as in memory, the V^T fragments come from the transposing LDS read.
// A tile of 64 keys takes a lone wave 1430 cycles, 830 of them vector issue: kReadAll, all K fragments are read before the first
// product and all V^T fragments before the softmax (read where they are used, each product waits for its own read: 1580).  us
// a launch, head of 1920 tokens and 32 columns, one workgroup a unit 23.1 -> 21.3; a step of 2 x 4200 tokens, 5-40 %, 8 heads
// of 32, 23.0 -> 21.7, 8 images 32.7 -> 31.5 (which form where: where the kernel is launched).  The scores of the next tile beside the exponentials, from a
// ring of three tiles, without a spill in the loop: 23.1 -> 25.5, 8 images 34.6 -> 39.
template <int DH, int BN>
struct TiledLds {
  static constexpr int RS = DH + 8;
  __attribute__((aligned(16))) __bf16 Ks[2][BN * RS];
  __attribute__((aligned(16))) __bf16 Vs[2][BN * RS];
};
constexpr int kTiledBN = 64;

// The workgroup's work on queries [q0, q0 + 32 NW) of head h of segment seg (q0 < seg.nq).
template <int DH, int NW, int READS, int GATHER>
__device__ __forceinline__ void
tiled_attention(TiledLds<DH, kTiledBN>& lds, const Segment seg, int h, int q0, const __bf16* __restrict__ q,
                const __bf16* __restrict__ k, const __bf16* __restrict__ v, long qs, long ks, long vs, int H,
                const float* __restrict__ v_scores, float scale_log2, __bf16* __restrict__ out, float* __restrict__ lse,
                long lse_stride, const Scatter& sc) {
  constexpr int RS = DH + 8, BN = kTiledBN, GSB = BN / 32;
  auto& Ks = lds.Ks;
  auto& Vs = lds.Vs;
  static_assert(2 * BN >= 32 * NW, "the K buffers double as the output staging tile");
  const long C = (long)H * DH;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, l32 = lane & 31, hh = lane >> 5;
  const int qi = q0 + wv * 32 + l32;
  const bool wave_live = q0 + wv * 32 < seg.nq;
  const bool q_ok = qi < seg.nq;

  const int32_t* gi = gather_base<GATHER>(sc, seg.row0);
  const long q_src = q_ok ? source_row(gi, seg.row0, qi) : 0;   // (gathered: an index load, issued first)
  const int y_row = GATHER ? (int)q_src : sc.y != nullptr && q_ok ? sc.gather_idx[seg.row0 + qi] : 0;
  PairStage<DH, 64 * NW, BN, GATHER != 0, GATHER != 0> stage(threadIdx.x);
  stage.gi = gi;
  stage.last = max(seg.nk - 1, 0);
  stage.source(0, k + h * DH, ks, seg.row0);
  stage.source(1, v + h * DH, vs, seg.row0);
  float gate[decltype(stage)::CPT] = {};
  auto load_tile = [&](int kt) {                                // (then the index of the one after it)
    stage.load(kt);
    if (is_gated(GATHER)) {
#pragma unroll
      for (int t = 0; t < decltype(stage)::CPT; ++t) gate[t] = v_scores[stage.idx[t]];
    }
    stage.index(kt + BN);
  };
  auto store_tile = [&](int buf, auto clear) {
    if (is_gated(GATHER)) stage.template store_gated<clear>(Ks[buf], Vs[buf], gate);
    else stage.template store<clear>(Ks[buf], Vs[buf]);
  };
  stage.index(0);
  load_tile(0);
  bf16x8 qf[DH / 16];
  load_q_frags<DH>(q + q_src * qs + h * DH, q_ok, hh, qf);
  FwdAcc<DH> acc;
  acc.init();
  store_tile(0, std::true_type{});
  __syncthreads();

  const int nt = (seg.nk + BN - 1) / BN;
  walk_tiles(nt, [&](int t, auto at) {
    constexpr bool last = decltype(at)::value == kTileLast;
    const int buf = t & 1, kt = t * BN;
    if (!last) load_tile(kt + BN);
    if (wave_live) {
      floatx16 s[GSB];
      fwd_scores<DH, RS, GSB, !last, READS != kReadLate>(Ks[buf], 0, seg.nk - kt, qf, s, l32, hh);
      fwd_softmax_pv<DH, 0, GSB, !last, READS>(s, Vs[buf], 0, 0, seg.nk - kt, acc, scale_log2, l32, hh);
    }
    if (!last) store_tile(buf ^ 1, std::bool_constant<decltype(at)::value == kTileBeforeLast>{});
    __syncthreads();
  });
  // every wave is past its last read of the K buffers
  __bf16* parked = &Ks[0][0] + wv * 32 * RS;
  if (wave_live) {
    fwd_park<DH, RS>(acc, q_ok, seg.nk > 0, parked, lse != nullptr ? lse + h * lse_stride + seg.row0 + qi : nullptr,
                     l32, hh);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    fwd_flush<DH, RS, GATHER == kFwdGatedD>(parked, out, sc, y_row, seg.row0 + q0 + wv * 32, h, C, min(32, seg.nq - q0 - wv * 32),
                                           lane, sc.dvec + h * lse_stride);
  }
}

// Workgroups [0, ntile) take query blocks, the rest fill y's bypassing rows while those run.
//   up to 64 segments and 64 pairs per XCD: live blocks only, longest segment first (live_order); a launch has
//     at most as many workgroups as are resident together, and number g of an XCD's G takes blocks g,
//     2 G - 1 - g, 2 G + g, ...: the order is found once per workgroup;
//   up to 256 segments: live blocks first, longest segment first, one per workgroup (class_tile_block; 122 x 480
//     tokens, 6-48 %, 11 heads of 64: 114 us with block qb of every pair in turn, 55 so);
//   otherwise (and for padded batches) block qb of every (segment, head) pair in turn.
template <int DH>
struct TiledShared {
  TiledLds<DH, kTiledBN> lds;
  int s_cu[2 * kLptMaxB + 1];
  int s_pick;
};
template <int DH, int NW, int READS, int GATHER>
__device__ __forceinline__ void tiled_block(TiledShared<DH>& sh, const FwdArgs& a, unsigned block, unsigned blocks) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, H = a.H, B = a.B;
  const Scatter& sc = a.sc;
  auto attend = [&](const Segment& seg, int h, int q0) {
    tiled_attention<DH, NW, READS, GATHER>(sh.lds, seg, h, q0, a.q, a.k, a.v, a.qs, a.ks, a.vs, H, a.v_scores, a.scale_log2,
                                        a.out, a.lse, a.lse_stride, sc);
  };
  if ((int)block >= a.ntile) {
    const long rows = sc.flat ? (long)sc.N : (long)B * sc.N;
    const long units = (long)(blocks - a.ntile) * NW, u = (long)(block - a.ntile) * NW + wv, per = (rows + units - 1) / units;
    scatter_fill_rows<__bf16>(sc, min(rows, u * per), min(rows, (u + 1) * per), (long)H * DH, lane);
    return;
  }
  if (a.key_lens == nullptr && live_tiles_apply(H, B)) {
    const int xcd = block & 7, G = a.ntile >> 3, g = there_and_back(block >> 3, G);
    int(*order)[64] = reinterpret_cast<int(*)[64]>(sh.s_cu);
    static_assert(sizeof(sh.s_cu) >= 5 * 64 * sizeof(int), "holds the order");
    if (wv == 0) {
      const LiveOrder o = live_order(xcd, H, B, a.cu, 32 * NW, a.nqb);
      order[0][lane] = o.len;
      order[1][lane] = o.start;
      order[2][lane] = o.img;
      order[3][lane] = o.nb;
      order[4][lane] = o.incl;
    }
    __syncthreads();
    for (int round = 0;; ++round) {
      const LiveOrder o = {order[0][lane], order[1][lane], order[2][lane], order[3][lane], order[4][lane]};
      const LiveTile lt = live_pick(o, xcd, round * G + (round & 1 ? G - 1 - g : g), H);
      if (!lt.valid) return;
      if (round > 0) __syncthreads();                       // the parked rows are written
      // More live blocks than workgroups: the longer segments, which began the launch, also end it, so they go first where a
      // SIMD's waves compete (32 x 4200 tokens, 5-40 %, 8 heads of 32: 63.2 -> 61.0 us, 48 images 115 -> 106; 8 images, two
      // workgroups a unit: 23.0 -> 23.5, so not there).
      if (__builtin_amdgcn_readlane(o.incl, 63) > G) {
        if (4 * lt.len > 3 * lt.longest) __builtin_amdgcn_s_setprio(3);
        else if (2 * lt.len > lt.longest) __builtin_amdgcn_s_setprio(2);
        else if (4 * lt.len > lt.longest) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
      }
      attend({lt.row0, lt.len, lt.len}, lt.h, lt.qb * (32 * NW));
    }
  }
  if (a.key_lens == nullptr && B <= kLptMaxB) {
    const LiveTile lt = class_tile_block<1>(block & 7, block >> 3, H, B, a.cu, 32 * NW, a.nqb,
                                            reinterpret_cast<LiveTile*>(sh.s_cu));
    if (lt.valid) attend({lt.row0, lt.len, lt.len}, lt.h, lt.qb * (32 * NW));
    return;
  }
  const TileId tile_id = xcd_tile_at(block & 7, block >> 3, a.nqb, H, B);
  if (!tile_id.valid) return;
  const Segment seg = lpt_segment<64 * NW>(tile_id.rank, B, a.cu, a.key_lens, a.n_pad, sh.s_cu, &sh.s_pick);
  const int q0 = tile_id.qb * (32 * NW);
  if (q0 < seg.nq) attend(seg, tile_id.h, q0);
}

template <int DH, int NW, int READS, int GATHER>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(DH == 64 || READS == kReadAll ? 3 : 4)))
attn_fwd_bf16_tiled_kernel(const FwdArgs a) {
  __shared__ TiledShared<DH> sh;
  // (at head dim 64 the form that leaves D has no register for an early read: 32 x 400 tokens, 6 heads, a training step, some |
  // late 62.8 | 61.4 us)
  tiled_block<DH, NW, DH == 64 && GATHER == kFwdGatedD ? kReadLate : READS, GATHER>(sh, a, blockIdx.x, gridDim.x);
}

// Short segments.  A work unit is 32 queries of one (image, head); SPLIT waves share it, each taking every SPLIT-th step of
// STEP keys.  A wave streams its keys' K and V rows through a private LDS tile (coalesced 16-byte row loads, its next step's
// rows already in flight in registers; KREGS: V alone), reads K fragments back as MFMA A operands and V fragments through the transposing
// LDS read, and keeps the online softmax state in registers; no barrier until the waves of a unit merge at the end.  Work
// units are small (<= n/32 steps each), so the load spreads over all SIMDs instead of concentrating a heavy (image,
// head) on one compute unit.
template <int DH, int STEP>
struct WaveLds {
  static constexpr int RS = DH + 8;
  __attribute__((aligned(16))) __bf16 Ks[STEP * RS];
  __attribute__((aligned(16))) __bf16 Vs[STEP * RS];
};

// The sums of waves 1 .. SPLIT - 1 of a unit go to the first one through LDS (room: 64 (DH / 2 + 2) floats a wave at
// lds + part * stride).  All waves call it; true for the first.  A wave that had no keys counts with weight 0.
template <int DH, int SPLIT>
__device__ __forceinline__ bool merge_parts(FwdAcc<DH>& acc, int part, bool have_keys, void* lds, int stride, int lane) {
  if (part > 0) {
    floatx4* o = reinterpret_cast<floatx4*>(static_cast<char*>(lds) + part * stride);
    float* ml = reinterpret_cast<float*>(o + DH / 8 * kWave);
#pragma unroll
    for (int g = 0; g < DH / 8; ++g)
      o[g * kWave + lane] = floatx4{acc.o[g / 4][4 * (g % 4)], acc.o[g / 4][4 * (g % 4) + 1], acc.o[g / 4][4 * (g % 4) + 2],
                                    acc.o[g / 4][4 * (g % 4) + 3]};
    ml[lane] = acc.m;
    ml[kWave + lane] = acc.l;
  }
  __syncthreads();
  if (part > 0) return false;
  if (!have_keys) return true;
  float m[SPLIT], m_all = acc.m;
#pragma unroll
  for (int i = 1; i < SPLIT; ++i) {
    m[i] = reinterpret_cast<const float*>(static_cast<const char*>(lds) + i * stride)[DH / 8 * kWave * 4 + lane];
    m_all = fmaxf(m_all, m[i]);
  }
  const float a = __builtin_amdgcn_exp2f(acc.m - m_all);
  acc.m = m_all;
  acc.l *= a;
#pragma unroll
  for (int d = 0; d < DH / 32; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc.o[d][r] *= a;
#pragma unroll
  for (int i = 1; i < SPLIT; ++i) {
    const floatx4* o = reinterpret_cast<const floatx4*>(static_cast<const char*>(lds) + i * stride);
    const float w = __builtin_amdgcn_exp2f(m[i] - m_all);
    acc.l = fmaf(reinterpret_cast<const float*>(o + DH / 8 * kWave)[kWave + lane], w, acc.l);
#pragma unroll
    for (int g = 0; g < DH / 8; ++g) {
      const floatx4 f = o[g * kWave + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc.o[g / 4][4 * (g % 4) + e] = fmaf(f[e], w, acc.o[g / 4][4 * (g % 4) + e]);
    }
  }
  return true;
}

// The work of wave `part` on queries [q0, q0 + 32) of head h of segment seg (q0 < seg.nq); lds: the unit's tiles, one a wave.
template <int DH, int STEP, int GATHER, int SPLIT>
__device__ __forceinline__ void
wave_attention(WaveLds<DH, STEP>* lds, int part, const Segment seg, int h, int q0, const __bf16* __restrict__ q,
               const __bf16* __restrict__ k, const __bf16* __restrict__ v, long qs, long ks, long vs, int H,
               const float* __restrict__ v_scores, float scale_log2, __bf16* __restrict__ out, float* __restrict__ lse, long lse_stride,
               const Scatter& sc) {
  constexpr int RS = DH + 8, KK = DH / 16, CPR = DH / 8;
  constexpr int NSB = STEP / 32;                 // 32-key sub-tiles per step (one softmax update)
  constexpr int LPL = STEP * CPR / 64;           // 16-byte loads per lane per tensor per step
  // Rows named by an index: K goes from memory to registers as the A operand of the scores (a lane holds its chunks of key
  // l32 of each sub-tile), not through LDS, and the V^T fragments are read before the softmax: one LDS round trip fewer on a
  // wave's chain.  us a step, before -> now: 64 x 196 tokens, 6 heads of 64, from the mask 15.9 -> 15.3 (128 images 23.4 | 23.4),
  // containers of 49 tokens, 12 heads of 32, 18.5 -> 18.3.  Rows of whole lines are cheaper to load where all SIMDs are busy with
  // products: packed, 128 x 196 tokens, 12 heads of 64, forward and backward, 356.6 -> 360.9, gated, 64 images, 80.6 -> 81.5.
  // Steps of 64 keys have no registers for it (head dim 64: one wave a SIMD instead of two, 64 x 196 tokens, 6 heads, through
  // the index 21.1 -> 23.9; head dim 32, 12 heads: two instead of three, 20.0 -> 21.2).
  constexpr bool KREGS = GATHER == kFwdGathered && STEP == 32;
  if (SPLIT == 1) part = 0;                      // (known here: the loop and the tiles of the one-wave form depend on it)
  __bf16 *Ks = lds[part].Ks, *Vs = lds[part].Vs;
  const long C = (long)H * DH;
  const int lane = threadIdx.x & 63, l32 = lane & 31, hh = lane >> 5;
  const int qi = q0 + l32;
  const bool q_ok = qi < seg.nq;
  const __bf16* kh = k + h * DH;
  const __bf16* vh = v + h * DH;

  // lane -> (row, chunk) of the step's tile: 8 (Dh 64) or 4 (Dh 32) lanes cover one row
  bf16x8 kreg[LPL], vreg[LPL];
  float gate[LPL] = {};
  const int32_t* gi = gather_base<GATHER>(sc, seg.row0);
  int tok_rows[LPL];                              // gathered rows only: token rows of the next gload
  int k_rows[NSB];                                // KREGS: of this lane's keys
  const int last_key = max(seg.nk - 1, 0);
  int kt_next = 0;                                // first key of the step the next gload fetches
  const int c = lane % CPR, lrow = lane / CPR;
  const uint32_t koff = (uint32_t)lrow * (uint32_t)ks + c * 8, voff = (uint32_t)lrow * (uint32_t)vs + c * 8;
  auto iload = [&](int kt) {                      // issued one step ahead of the row loads that use it
    kt_next = kt;
    if constexpr (KREGS) {
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb) k_rows[sb] = gi[min(kt + sb * 32 + l32, last_key)];
    }
    if (GATHER) {
#pragma unroll
      for (int t = 0; t < LPL; ++t) {
        const int r = kt + lrow + t * (64 / CPR);
        if (r < seg.nk) tok_rows[t] = gi[r];
      }
    }
  };
  auto gload = [&]() {                            // rows past the segment: zero, KREGS: the last K row (their scores are masked)
    if constexpr (KREGS) {
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
          kreg[sb * KK + kk] = *reinterpret_cast<const bf16x8*>(kh + row_offset(k_rows[sb], ks) + hh * 8 + kk * 16);
    }
#pragma unroll
    for (int t = 0; t < LPL; ++t) {
      if (!KREGS) kreg[t] = zero_bf16x8();
      vreg[t] = zero_bf16x8();
      if (kt_next + lrow + t * (64 / CPR) < seg.nk) {
        const __bf16 *kp, *vp;
        if (GATHER) {
          kp = kh + row_offset(tok_rows[t], ks) + c * 8;
          vp = vh + row_offset(tok_rows[t], vs) + c * 8;
        } else {
          const long r = seg.row0 + kt_next + t * (64 / CPR);    // uniform: the lane's part is koff / voff
          kp = kh + r * ks + koff;
          vp = vh + r * vs + voff;
        }
        if (!KREGS) kreg[t] = *reinterpret_cast<const bf16x8*>(kp);
        vreg[t] = *reinterpret_cast<const bf16x8*>(vp);
        if (is_gated(GATHER)) gate[t] = v_scores[tok_rows[t]];
      }
    }
  };
  auto lstore = [&]() {
#pragma unroll
    for (int t = 0; t < LPL; ++t) {
      const int i = lane + 64 * t, r = i / CPR, c = i % CPR;
      if (!KREGS) *reinterpret_cast<bf16x8*>(&Ks[r * RS + c * 8]) = kreg[t];
      *reinterpret_cast<bf16x8*>(&Vs[r * RS + c * 8]) =
          is_gated(GATHER) ? scale_row(vreg[t], sigmoidf_dev(gate[t])) : vreg[t];
    }
  };

  const int first = part * STEP;
  const long q_src = q_ok ? source_row(gi, seg.row0, qi) : 0;   // (gathered: an index load, issued first, so that
  iload(first);                                                  // its wait is the one the first row loads need anyway)
  gload();
  iload(first + SPLIT * STEP);
  bf16x8 qf[KK];
  load_q_frags<DH>(q + q_src * qs + h * DH, q_ok, hh, qf);
  // the row of y of this lane's query: the row it was read from, or fetched now, when nothing waits for it yet
  const int y_row = GATHER ? (int)q_src : sc.y != nullptr && q_ok ? sc.gather_idx[seg.row0 + qi] : 0;
  FwdAcc<DH> acc;
  acc.init();

  for (int kt = first; kt < seg.nk; kt += SPLIT * STEP) {
    // scores of the step: S^T = K Q^T, NSB 32-key sub-tiles, one softmax update for all
    const int rem = seg.nk - kt;
    floatx16 s[NSB];
    if constexpr (KREGS) {
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[sb][r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) s[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kreg[sb * KK + kk], qf[kk], s[sb], 0, 0, 0);
      }
    }
    lstore();                                     // this step's rows: registers -> LDS
    if (kt + SPLIT * STEP < seg.nk) {
      gload();                                    // next step's rows: in flight during the math
      iload(kt + 2 * SPLIT * STEP);
    }
    if constexpr (KREGS) {
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb)
        if (rem - sb * 32 < 32) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (sb * 32 + acc_row(r, hh) >= rem) s[sb][r] = -INFINITY;
        }
    } else {
      fwd_scores<DH, RS, NSB, false>(Ks, 0, rem, qf, s, l32, hh);
    }
    fwd_softmax_pv<DH, 0, NSB, false, KREGS ? kReadAll : kReadLate>(s, Vs, 0, 0, rem, acc, scale_log2, l32, hh);
  }

  if constexpr (SPLIT > 1)
    if (!merge_parts<DH, SPLIT>(acc, part, seg.nk > 0, lds, sizeof(WaveLds<DH, STEP>), lane)) return;
  // output: park the 32 x DH tile in the (now free) K tile, then write whole rows
  fwd_park<DH, RS>(acc, q_ok, seg.nk > 0, Ks, lse != nullptr ? lse + h * lse_stride + seg.row0 + qi : nullptr, l32,
                   hh);
  fwd_flush<DH, RS, GATHER == kFwdGatedD>(Ks, out, sc, y_row, seg.row0 + q0, h, C, min(32, seg.nq - q0), lane,
                                         sc.dvec + h * lse_stride);
}

// Waves a unit.  One wave a unit lives 2 us + 0.8 us for every 32 keys + 1.5 us; where the units do not fill the chip (half
// of them have queries) that chain is the launch, so two waves share it, the merge costing 0.3 us.  With more units the
// waves of those without queries take the others' slots.  us a step, 196 tokens an image, 6 heads of 64, two launches,
// 1 / 2 / 4 waves: 8 images (336 units) 11.2 / 9.3 / 9.7, 16 images 12.0 / 10.0 / 10.5, 32 images (1344) 13.0 / 11.8 / 14.3,
// 64 images 15.9 / 16.5 / 20.5; 32 x 256 tokens, 6 heads of 64 (1536) 15.9 / 14.1.  Head dim 32, 6 heads: 18 x 256 tokens (864)
// 11.6 / 10.9, 32 x 256 (1536) 12.7 / 12.5, and beside other calls of a launch group, training, 100.0 / 101.4.
// Segments of up to 3 steps are not worth a merge.  Two waves add a row's keys in another order than one, so an image's bits are
// the same in any two calls on one side of this line, and differ by rounding across it.
static int unit_waves(int Dh, int nqb, long units) { return nqb >= 4 && units <= (Dh == 64 ? 1536 : 1024) ? 2 : 1; }

template <int SPLIT, int DH, int STEP, int GATHER>
__global__ void __launch_bounds__(64 * SPLIT) __attribute__((amdgpu_waves_per_eu(STEP == 32 ? 3 : 1)))
attn_fwd_bf16_wave_kernel(const FwdArgs a) {
  __shared__ WaveLds<DH, STEP> lds[SPLIT];
  const TileId tile_id = xcd_tile(a.nqb, a.H, a.B);
  if (!tile_id.valid) return;
  const int h = tile_id.h, img = tile_id.rank;
  const Segment seg = segment_of(img, a.cu, a.key_lens, a.n_pad);
  const long C = (long)a.H * DH;
  // this unit's share of the image's bypassing tokens: at once if it has no queries, else last
  const FillRange fr = fill_range(a.sc, img, a.B, tile_id.qb, a.nqb);
  const int q0 = tile_id.qb * 32;
  if (q0 < seg.nq)
    wave_attention<DH, STEP, GATHER, SPLIT>(lds, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), seg, h, q0, a.q, a.k, a.v, a.qs, a.ks, a.vs, a.H, a.v_scores,
                                            a.scale_log2, a.out, a.lse, a.lse_stride, a.sc);
  if (a.sc.y != nullptr) scatter_fill<__bf16, DH>(a.sc, fr.b, fr.t0, fr.t1, h, C, threadIdx.x, 64 * SPLIT);
}

// The work units driven by the selection mask itself: no packing launch precedes this
// kernel.  Every wave reads its image's N <= 256 mask bytes, ranks the survivors with ballots and
// writes their token rows, in order, to a list in LDS: exactly the image's part of gather_idx, so
// wave_attention runs on it as on gathered rows (packed position j of the image = row list[j] of
// q, k, v and of y), and the bypass fill tests the mask byte instead of inv_pos.  Costs four byte
// loads and four ballots per wave where the other forms cost a kernel launch.
template <int DH, int STEP, int SPLIT>
struct MaskLds {
  WaveLds<DH, STEP> kv[SPLIT];
  int32_t list[256];
};
// Unit j of XCD xcd (N <= 256 tokens per image, mask and fill of y: a.sc), wave `part` of it
template <int DH, int STEP, int SPLIT>
__device__ __forceinline__ void mask_unit(MaskLds<DH, STEP, SPLIT>& lds, const FwdArgs& a, int xcd, int j, int part) {
  if (SPLIT == 1) part = 0;
  const TileId tile_id = xcd_tile_at(xcd, j, a.nqb, a.H, a.B);
  if (!tile_id.valid) {
    if (SPLIT > 1) __syncthreads();
    return;
  }
  const int h = tile_id.h, img = tile_id.rank, lane = threadIdx.x & 63, N = a.sc.N;
  const long tok0 = (long)img * N;
  int n = 0;                                       // survivors of the image so far
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int t = lane + 64 * i;
    const bool sel = t < N && a.sc.mask[tok0 + t] != 0;
    const uint64_t bal = __ballot(sel);
    if (sel) lds.list[n + lanes_below(bal)] = (int32_t)(tok0 + t);      // (every wave of the unit writes the same list)
    n += __popcll(bal);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const Segment seg = {0, n, n};                   // packed rows numbered inside the image: row j <-> list[j]
  Scatter scl = a.sc;
  scl.gather_idx = lds.list;
  const long C = (long)a.H * DH;
  const FillRange fr = fill_range(a.sc, img, a.B, tile_id.qb, a.nqb);
  const int q0 = tile_id.qb * 32;
  if (q0 < n)
    wave_attention<DH, STEP, kFwdGathered, SPLIT>(lds.kv, part, seg, h, q0, a.q, a.k, a.v, a.qs, a.ks, a.vs, a.H, a.v_scores,
                                                  a.scale_log2, nullptr, nullptr, 0, scl);
  else if (SPLIT > 1) __syncthreads();             // (the workgroup's other unit merges)
  scatter_fill<__bf16, DH>(a.sc, fr.b, fr.t0, fr.t1, h, C, lane + 64 * part, 64 * SPLIT);
}

template <int DH, int STEP, int SPLIT>
__global__ void __launch_bounds__(64 * SPLIT) __attribute__((amdgpu_waves_per_eu(3)))
attn_fwd_bf16_wave_mask_kernel(const FwdArgs a) {
  __shared__ MaskLds<DH, STEP, SPLIT> lds;
  mask_unit<DH, STEP, SPLIT>(lds, a, blockIdx.x & 7, blockIdx.x >> 3, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// The same work units, dealt to the compute units by weight (batches of up to 64 images, one
// per lane).  All one-wave workgroups of the launch are resident at once and workgroup j of
// an XCD runs on compute unit j % 32 (the hardware id register says so), so which units get
// the long segments is decided by the numbering alone; numbered blindly, the unluckiest SIMDs
// end a third later than the median.  Here every wave ranks the images by their number of
// 32-key steps (9 classes, one ballot each; images of a class in index order), the (image,
// head) pairs of that ranking are dealt to the XCDs in snake order (an XCD's L2 still holds
// all blocks of its pairs), the XCD's live query blocks are listed heaviest first, and the
// m-th workgroup of a unit takes block r = 32 m + (unit, or 31 - unit for odd m).  Workgroups
// past the live blocks only fill; the bypassing rows of y are shared evenly by all.
// No tables are needed: with the pairs sorted by
// class, class c holds the ranked images [A_c, A_c + n_c) (n_c from one ballot), hence the
// pairs [A_c H, (A_c + n_c) H), of which this XCD owns a count with a closed form; every pair
// of class c has exactly c live blocks.  Walking the 9 classes with scalar arithmetic finds
// the class, the pair and the block of number r; the image is the k-th set bit of the class
// ballot and its bounds come by readlane.
// Block number r of XCD x -> its segment, head and first query (live = false: past the live
// blocks).  QB = queries per block; a segment's class is its number of blocks.  Every wave of
// the workgroup computes the same answer from its own ballots.
struct LptBlock {
  Segment seg;
  int h, q0;
  bool live;
};
template <int QB>
__device__ __forceinline__ LptBlock lpt64_block(const int32_t* __restrict__ cu, const int32_t* __restrict__ key_lens,
                                                int n_pad, int B, int H, int nqb, int x, int r) {
  const int lane = threadIdx.x & 63;
  const bool padded = key_lens != nullptr;
  int start = 0, len = 0, cls = -1;
  if (lane < B) {
    if (padded) {
      start = lane * n_pad;
      len = min(max(key_lens[lane], 0), n_pad);
    } else {
      start = cu[lane];
      len = cu[lane + 1] - start;
    }
    cls = min((max(len, 0) + QB - 1) / QB, nqb);
  }
  LptBlock blk = {{0, 0, 0}, 0, 0, false};
  int ranked = 0, tiles = 0, g0 = 0;             // images, live blocks, this XCD's pairs of the heavier classes
  for (int c = nqb; c >= 0; --c) {
    const uint64_t bal = __ballot(cls == c);
    const int n_c = __popcll(bal);
    const int per_pair = padded ? nqb : c;
    const int pairs_c = pairs_below((ranked + n_c) * H, x) - pairs_below(ranked * H, x);
    const int tiles_c = pairs_c * per_pair;
    if (r < tiles + tiles_c) {
      const int idx = r - tiles, g = g0 + idx / per_pair;
      const int p = 8 * g + ((g & 1) ? 7 - x : x);
      const int img = kth_set_bit(bal, p / H - ranked);
      blk.h = p % H;
      blk.q0 = (idx % per_pair) * QB;
      blk.seg.row0 = __builtin_amdgcn_readlane(start, img);
      blk.seg.nk = __builtin_amdgcn_readlane(len, img);
      blk.seg.nq = padded ? n_pad : blk.seg.nk;
      blk.live = blk.q0 < blk.seg.nq;
      break;
    }
    tiles += tiles_c;
    g0 += pairs_c;
    ranked += n_c;
  }
  return blk;
}
// the grid of such a launch: 8 XCDs x 32 units x enough rounds for all blocks of the XCD with most pairs
static unsigned lpt64_grid(int B, int H, int nqb) {
  const long g8 = ((long)B * H + 7) / 8;
  return (unsigned)(8 * 32 * ((g8 * nqb + 31) / 32));
}

// Compiled for three waves per SIMD (168 registers at head dim 64, no spills): a ViT-B-shaped
// batch has ~2800 live waves for 1024 SIMDs and then runs in one round instead of two.
template <int DH, int STEP, int GATHER, int SPLIT>
__device__ __forceinline__ void lpt64_unit(WaveLds<DH, STEP>* lds, const FwdArgs& a, int x, int j, int units, int part) {
  if (SPLIT == 1) part = 0;
  const int unit = j & 31, m = j >> 5;
  const LptBlock blk = lpt64_block<32>(a.cu, a.key_lens, a.n_pad, a.B, a.H, a.nqb, x, m * 32 + ((m & 1) ? 31 - unit : unit));
  if (blk.live)
    wave_attention<DH, STEP, GATHER, SPLIT>(lds, part, blk.seg, blk.h, blk.q0, a.q, a.k, a.v, a.qs, a.ks, a.vs, a.H,
                                            a.v_scores, a.scale_log2, a.out, a.lse, a.lse_stride, a.sc);
  else if (SPLIT > 1) __syncthreads();           // (the workgroup's other unit merges)
  if (a.sc.y != nullptr) {
    const long rows = a.sc.flat ? (long)a.sc.N : (long)a.B * a.sc.N, waves = (long)units * SPLIT, per = (rows + waves - 1) / waves,
               u = (8L * j + x) * SPLIT + part;
    scatter_fill_rows<__bf16>(a.sc, min(rows, u * per), min(rows, (u + 1) * per), (long)a.H * DH, threadIdx.x & 63);
  }
}
template <int SPLIT, int DH, int STEP, int GATHER>
__global__ void __launch_bounds__(64 * SPLIT) __attribute__((amdgpu_waves_per_eu(3)))
attn_fwd_bf16_wave_lpt64_kernel(const FwdArgs a) {
  __shared__ WaveLds<DH, STEP> lds[SPLIT];
  lpt64_unit<DH, STEP, GATHER, SPLIT>(lds, a, blockIdx.x & 7, blockIdx.x >> 3, gridDim.x, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
}

// Several calls in one launch (launch groups, head dim 32): the tiled blocks of those with more than 256 tokens
// per image, four of the one-wave units of the others (kFwdGathered: by their mask) per workgroup.  The blocks that attend
// come first, of all calls, and then those that only fill rows of y: a call after one with 1024 of these started its longest
// segments 5 us late (four stages of 16 x 3136 tokens 28.9 -> 28.0 us, their training forward 32.5 -> 31.0).
__device__ __forceinline__ MemberBlock work_first(const Members<FwdArgs>& m, unsigned block) {
  unsigned work[kGroupMax], all[kGroupMax];
#pragma unroll
  for (int s = 0; s < kGroupMax; ++s) {
    all[s] = m.end[s] - (s > 0 ? m.end[s - 1] : 0u);
    work[s] = m.a[s].ntile > 0 ? min((unsigned)m.a[s].ntile, all[s]) : all[s];
  }
  int s = 0;
  for (; s < kGroupMax && block >= work[s]; ++s) block -= work[s];
  if (s < kGroupMax) return {s, block, all[s]};
  for (s = 0; s < kGroupMax - 1 && block >= all[s] - work[s]; ++s) block -= all[s] - work[s];
  return {s, work[s] + block, all[s]};
}
// Four waves a SIMD: the workgroups beyond the three a unit that walk the longest segments are those of the other calls (four
// stages of 16 x 3136 tokens 40.2 us a step, with three 42.3).  128 registers hold all of a tile's reads early but for gated
// rows, of which they hold some: all with spills | late | some, a training step of four stages of 16 x 3136 tokens 133.2 | 131.1 |
// 131.1, of four images 73.8 | 73.8 | 73.4, of one 60.6 | 60.9 | 60.6; forward, all | late, 4 x 3136 30.1 | 31.2.
template <int FORM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
attn_fwd_bf16_group_kernel(const Members<FwdArgs> m) {
  constexpr int DH = 32, STEP = 32;
  constexpr int READS = is_gated(FORM) ? kReadSome : kReadAll;
  __shared__ union {
    TiledShared<DH> tiled;
    MaskLds<DH, STEP, 1> wave[4];
    MaskLds<DH, STEP, 2> pair[2];
  } sh;
  const MemberBlock mb = work_first(m, blockIdx.x);
  const FwdArgs& a = m.a[mb.s];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (a.ntile > 0) tiled_block<DH, 4, READS, FORM>(sh.tiled, a, mb.block, mb.blocks);
  else if (a.waves == 2) {
    const int j = (mb.block >> 3) * 2 + (wv >> 1);
    if constexpr (FORM == kFwdGathered) mask_unit<DH, STEP, 2>(sh.pair[wv >> 1], a, mb.block & 7, j, wv & 1);
    else lpt64_unit<DH, STEP, FORM, 2>(sh.pair[wv >> 1].kv, a, mb.block & 7, j, mb.blocks * 2, wv & 1);
  } else {
    const int j = (mb.block >> 3) * 4 + wv;
    if constexpr (FORM == kFwdGathered) mask_unit<DH, STEP, 1>(sh.wave[wv], a, mb.block & 7, j, 0);
    else lpt64_unit<DH, STEP, FORM, 1>(sh.wave[wv].kv, a, mb.block & 7, j, mb.blocks * 4, 0);
  }
}

// Where call w of the same launch writes into the dy of call d (dy = y is the gradient of |y|^2 / 2), the launch cannot form
// the D of d: it would read dy too early, or while it is written.
static bool dy_apart(const FwdArgs& d, const FwdArgs& w, int Dh) {
  const size_t bytes = (size_t)d.lse_stride * d.H * Dh * sizeof(__bf16);
  const auto apart_from = [&](const void* p, size_t n) { return p == nullptr || apart(d.sc.dy, bytes, p, n); };
  const size_t rows = (size_t)w.lse_stride * w.H * Dh * sizeof(__bf16);
  return apart_from(w.sc.y, rows) && apart_from(w.out, rows) && apart_from(w.lse, (size_t)w.lse_stride * w.H * sizeof(float));
}
static void launch_dvec_of(const FwdArgs& d, int Dh, hipStream_t st) {
  launch_dvec(d.out, d.sc.dy, d.sc.gather_idx, d.cu, d.B, d.H, Dh, d.lse_stride, d.sc.dvec, st);
}

static thread_local Noted<FwdArgs> g_noted[kFwdForms];       // by form
void group_forget_attention() { for (auto& g : g_noted) g.n = 0; }
template <int FORM>
static void flush_form(Noted<FwdArgs>& noted, hipStream_t st) {
  if (noted.n == 0) return;
  Members<FwdArgs> m;
  const unsigned blocks = noted.members(m);
  hipLaunchKernelGGL((attn_fwd_bf16_group_kernel<FORM>), dim3(blocks), dim3(256), 0, st, m);
}
int group_flush_attention(hipStream_t st) {
  Noted<FwdArgs> with_d, after;                              // D in the launch; in one of its own after them all
  const Noted<FwdArgs>& d = g_noted[kFwdGatedD];
  for (int i = 0; i < d.n; ++i) {
    bool beside = true;
    for (const auto& g : g_noted)
      for (int j = 0; j < g.n; ++j) beside = beside && dy_apart(d.a[i], g.a[j], 32);
    if (int rc = (beside ? with_d : after).add("spa_group_end", d.a[i], d.blocks[i])) return rc;
  }
  const int late = after.n;
  g_noted[kFwdGatedD].n = 0;
  flush_form<kFwdPacked>(g_noted[kFwdPacked], st);
  flush_form<kFwdGathered>(g_noted[kFwdGathered], st);
  flush_form<kFwdGated>(g_noted[kFwdGated], st);
  flush_form<kFwdGatedD>(with_d, st);
  flush_form<kFwdGated>(after, st);
  for (int i = 0; i < late; ++i) launch_dvec_of(after.a[i], 32, st);
  return check_launch("spa_group_end");
}
// workgroups of four waves for so many units (8 XCDs)
static unsigned wave_groups(unsigned units, int waves) { return (units / 8 * waves + 3) / 4 * 8; }

// Short segments (every segment <= NKMAX keys).  ONE workgroup per (image, head): all K / V
// rows of the segment are staged once (each element is read from memory exactly once per
// head), one barrier, then wave w owns queries [32w, 32w+32) and walks the keys in LDS with
// no further synchronisation.  No workgroup is launched for nothing.
template <int DH, int NKMAX, int GATHER>
__global__ void __launch_bounds__(2 * NKMAX)
attn_fwd_bf16_whole_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                           const __bf16* __restrict__ v, long qs, long ks, long vs,
                           const int32_t* __restrict__ cu, const int32_t* __restrict__ key_lens, int n_pad,
                           int H, float scale_log2, __bf16* __restrict__ out, float* __restrict__ lse,
                           long lse_stride, Scatter sc) {
  constexpr int THREADS = 2 * NKMAX;                       // one wave per 32 queries
  constexpr int RS = DH + 8, TS = transposed_stride(NKMAX);
  constexpr int TILE = NKMAX < 128 ? NKMAX : 128;           // keys per softmax update
  constexpr int NSB = TILE / 32;
  __shared__ __attribute__((aligned(16))) __bf16 Ks[NKMAX * RS];
  __shared__ __attribute__((aligned(16))) __bf16 Vt[DH * TS];

  const int h = blockIdx.x;
  Segment seg = segment_of(blockIdx.y, cu, key_lens, n_pad);
  seg.nq = min(seg.nq, NKMAX);   // never index past the LDS tile, whatever cu_seqlens holds
  seg.nk = min(seg.nk, NKMAX);
  const long C = (long)H * DH;
  const FillRange fr = fill_range(sc, blockIdx.y, gridDim.y, 0, 1);
  if (seg.nq <= 0) {
    if (sc.y != nullptr) scatter_fill<__bf16, DH>(sc, fr.b, fr.t0, fr.t1, h, C, threadIdx.x, THREADS);
    return;
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, l32 = lane & 31, hh = lane >> 5;
  const int qi = wv * 32 + l32;
  const bool wave_live = wv * 32 < seg.nq;
  const bool q_ok = qi < seg.nq;

  const int32_t* gi = gather_base<GATHER>(sc, seg.row0);
  const int y_row = sc.y != nullptr && q_ok ? sc.gather_idx[seg.row0 + qi] : 0;
  KvStage<DH, THREADS, (NKMAX / 2) * (DH / 8), GATHER> stage;
  stage.index(gi, seg.row0, 0, seg.nk);
  stage.load(k + h * DH, v + h * DH, ks, vs);
  bf16x8 qf[DH / 16];
  load_q_frags<DH>(q + (q_ok ? source_row(gi, seg.row0, qi) : 0) * qs + h * DH, q_ok, hh, qf);
  FwdAcc<DH> acc;
  acc.init();
  stage.template store<RS, TS>(Ks, Vt, 0);
  __syncthreads();
  // the rows that bypass attention are filled by the waves that own no queries while the
  // others compute; if every wave has queries (few rows bypass then) all do it at the end
  const int live_threads = ((seg.nq + 31) / 32) * 64;
  if (!wave_live && sc.y != nullptr)
    scatter_fill<__bf16, DH>(sc, fr.b, fr.t0, fr.t1, h, C, threadIdx.x - live_threads, THREADS - live_threads);
  if (wave_live) {
    for (int kt = 0; kt < seg.nk; kt += TILE) {
      const int rem = seg.nk - kt;
      if (rem >= TILE) fwd_process_tile<DH, RS, TS, NSB, true>(Ks + kt * RS, Vt, kt, TILE, qf, acc, scale_log2, l32, hh);
      else fwd_process_tile<DH, RS, TS, NSB, false>(Ks + kt * RS, Vt, kt, rem, qf, acc, scale_log2, l32, hh);
    }
  }
  __syncthreads();                       // all waves are done reading K: its rows become the output tile
  __bf16* tile = Ks + wv * 32 * RS;
  if (wave_live)
    fwd_park<DH, RS>(acc, q_ok, seg.nk > 0, tile, lse != nullptr ? lse + h * lse_stride + seg.row0 + qi : nullptr,
                     l32, hh);
  __syncthreads();
  if (wave_live) fwd_flush<DH, RS>(tile, out, sc, y_row, seg.row0 + wv * 32, h, C, min(32, seg.nq - wv * 32), lane);
  if (sc.y != nullptr && live_threads >= THREADS)
    scatter_fill<__bf16, DH>(sc, fr.b, fr.t0, fr.t1, h, C, threadIdx.x, THREADS);
}

// ------------------------------------------------------------------------------- fp32
// One wave per (image, head, 32 queries) on v_mfma_f32_32x32x2_f32 (fp32 products and sums, twice the
// rate of the vector ALU), everything in registers: no LDS tile, no barrier.  The contraction order is
// free, so a lane (row l32 of the operand, half hh) simply holds the elements hh DH/2 .. of its K or Q
// row, S^T = K Q^T leaves 16 keys of one query in a lane, and these probabilities are the B operand of
// O^T += V^T P^T, register r against V row acc_row(r, hh), of which the 32 lanes of a half read 128
// consecutive bytes.  The rows of the next 32 keys are in flight during the math.  Bound by latency at
// the sizes it is used at (2 x 196 tokens, 60 selected each: 5.6 us; its predecessor, eight lanes per query with K / V tiles
// in LDS, took 12.5).
template <int DH, int SPLIT>
__global__ void __launch_bounds__(64 * SPLIT) __attribute__((amdgpu_waves_per_eu(2)))
attn_fwd_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                    const float* __restrict__ v, long qs, long ks, long vs, const int32_t* __restrict__ cu,
                    const int32_t* __restrict__ key_lens, int n_pad, int H, float scale,
                    float* __restrict__ out, float* __restrict__ lse, long lse_stride, Scatter sc, int B, int nqb) {
  constexpr int HD = DH / 2, DB = DH / 32;
  const TileId tile_id = xcd_tile(nqb, H, B);
  if (!tile_id.valid) return;
  const int h = tile_id.h, img = tile_id.rank, lane = threadIdx.x & 63, l32 = lane & 31, hh = lane >> 5;
  const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long C = (long)H * DH;
  // cu == key_lens == nullptr: no packing index exists; the wave derives the image's packing order from
  // its n_pad <= 256 mask bytes (see attn_fwd_bf16_wave_mask_kernel) and works on that list as on gathered rows
  __shared__ int32_t list[256];
  Segment seg;
  if (cu == nullptr && key_lens == nullptr) {
    const long tok0 = (long)img * n_pad;
    int n = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = lane + 64 * i;
      const bool sel = t < n_pad && sc.mask[tok0 + t] != 0;
      const uint64_t bal = __ballot(sel);
      if (sel) list[n + rank_in_ballot(bal)] = (int32_t)(tok0 + t);      // (every wave of the unit writes the same list)
      n += __popcll(bal);
    }
    __syncthreads();
    seg = {0, n, n};
    sc.gather_idx = list;
  } else {
    seg = segment_of(img, cu, key_lens, n_pad);
  }
  const FillRange fr = fill_range(sc, img, B, tile_id.qb, nqb);
  const int q0 = tile_id.qb * 32;
  if (q0 < seg.nq) {
    const int qi = q0 + l32;
    const bool q_ok = qi < seg.nq;
    const int32_t* gi = sc.gathered ? sc.gather_idx + seg.row0 : nullptr;
    const float* kh = k + h * DH + hh * HD;
    const float* vh = v + h * DH + l32;
    // key rows: lane l32 fetches key kt + l32 (past the segment: its last key, masked below)
    float kf[HD], vf[16][DB], kn[HD], vn[16][DB];
    auto key_row = [&](int kt) { return (int)source_row(gi, seg.row0, min(kt + l32, seg.nk - 1)); };
    auto fetch = [&](int row, float (&kd)[HD], float (&vd)[16][DB]) {
      const float* kp = kh + (long)row * ks;
#pragma unroll
      for (int i = 0; i < HD; i += 4) {
        const floatx4 t = *reinterpret_cast<const floatx4*>(kp + i);
        kd[i] = t[0]; kd[i + 1] = t[1]; kd[i + 2] = t[2]; kd[i + 3] = t[3];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float* vp = vh + (long)__shfl(row, acc_row(r, hh), kWave) * vs;
#pragma unroll
        for (int d = 0; d < DB; ++d) vd[r][d] = vp[d * 32];
      }
    };
    float qf[HD];
#pragma unroll
    for (int i = 0; i < HD; ++i) qf[i] = 0.f;
    const long q_src = source_row(gi, seg.row0, q_ok ? qi : 0);
    const int first = 32 * part;                         // keys first .. + 31, then every SPLIT-th 32
    int row = first < seg.nk ? key_row(first) : 0;
    if (q_ok) {
      const float* qp = q + q_src * qs + h * DH + hh * HD;
#pragma unroll
      for (int i = 0; i < HD; i += 4) {
        const floatx4 t = *reinterpret_cast<const floatx4*>(qp + i) * scale;
        qf[i] = t[0]; qf[i + 1] = t[1]; qf[i + 2] = t[2]; qf[i + 3] = t[3];
      }
    }
    floatx16 o[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
    float m = kNoScore, l = 0.f;
    if (first < seg.nk) {
      fetch(row, kf, vf);
      row = key_row(first + 32 * SPLIT);
    }
    for (int kt = first; kt < seg.nk; kt += 32 * SPLIT) {
      const int rem = seg.nk - kt;
      if (rem > 32 * SPLIT) {
        fetch(row, kn, vn);
        row = key_row(kt + 64 * SPLIT);
      }
      floatx16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
      for (int i = 0; i < HD; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[i], qf[i], s, 0, 0, 0);
      if (rem < 32) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (acc_row(r, hh) >= rem) {
            s[r] = -INFINITY;
#pragma unroll
            for (int d = 0; d < DB; ++d) vf[r][d] = 0.f;
          }
      }
      float mx = s[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
      const float m_new = fmaxf(m, max_across_halves(mx));
      const float alpha = expf(m - m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = expf(s[r] - m_new);
        l += s[r];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int d = 0; d < DB; ++d) o[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[r][d], s[r], o[d], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < HD; ++i) kf[i] = kn[i];
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int d = 0; d < DB; ++d) vf[r][d] = vn[r][d];
    }
    // the sums of waves 1 .. go to the first one (a wave that had no keys counts with weight 0)
    if constexpr (SPLIT > 1) {
      __shared__ float4 part_o[SPLIT - 1][DB * 4][kWave];
      __shared__ float part_ml[SPLIT - 1][2][kWave];
      if (part > 0) {
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            part_o[part - 1][d * 4 + g][lane] = float4{o[d][4 * g], o[d][4 * g + 1], o[d][4 * g + 2], o[d][4 * g + 3]};
        part_ml[part - 1][0][lane] = m;
        part_ml[part - 1][1][lane] = l;
      }
      __syncthreads();
      if (part == 0) {
        float m_all = m;
#pragma unroll
        for (int i = 0; i < SPLIT - 1; ++i) m_all = fmaxf(m_all, part_ml[i][0][lane]);
        const float a = seg.nk > 0 ? expf(m - m_all) : 1.f;
        l *= a;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[d][r] *= a;
        for (int i = 0; i < SPLIT - 1; ++i) {
          const float w = seg.nk > 0 ? expf(part_ml[i][0][lane] - m_all) : 0.f;
          l = fmaf(part_ml[i][1][lane], w, l);
#pragma unroll
          for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const float4 f = part_o[i][d * 4 + g][lane];
              o[d][4 * g] = fmaf(f.x, w, o[d][4 * g]);
              o[d][4 * g + 1] = fmaf(f.y, w, o[d][4 * g + 1]);
              o[d][4 * g + 2] = fmaf(f.z, w, o[d][4 * g + 2]);
              o[d][4 * g + 3] = fmaf(f.w, w, o[d][4 * g + 3]);
            }
        }
        m = m_all;
      }
    }
    const float l_tot = sum_across_halves(l);
    if (q_ok && part == 0) {
      const float inv = seg.nk > 0 ? 1.0f / l_tot : 0.f;
      float* op = out != nullptr ? out + (seg.row0 + qi) * C + h * DH + 4 * hh : nullptr;
      const long yoff = sc.y != nullptr ? (long)sc.gather_idx[seg.row0 + qi] * C + h * DH + 4 * hh : 0;
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int at = d * 32 + 8 * g;
          floatx4 t = {o[d][4 * g] * inv, o[d][4 * g + 1] * inv, o[d][4 * g + 2] * inv, o[d][4 * g + 3] * inv};
          if (op != nullptr) *reinterpret_cast<floatx4*>(op + at) = t;
          if (sc.y != nullptr) {
            if (sc.base != nullptr) t += *reinterpret_cast<const floatx4*>(static_cast<const float*>(sc.base) + yoff + at);
            __builtin_nontemporal_store(t, reinterpret_cast<floatx4*>(static_cast<float*>(sc.y) + yoff + at));
          }
        }
      if (lse != nullptr && hh == 0) lse[h * lse_stride + seg.row0 + qi] = seg.nk > 0 ? m + logf(l_tot) : -INFINITY;
    }
  }
  if (sc.y != nullptr) scatter_fill<float, DH>(sc, fr.b, fr.t0, fr.t1, h, C, threadIdx.x, 64 * SPLIT);
}

// ------------------------------------------------------------------------------- host
// fp32: four waves a unit where the units leave the chip idle and there are keys to split (2 x 196 tokens, 2 heads of 32,
// called again and again: 60 selected an image 6.9 -> 5.6 us, all 16.9 -> 7.6; the sums of an image then go by another order
// than in a larger batch)
template <class... Args>
static void launch_f32(int Dh, int B, int H, int nqb, hipStream_t st, Args... args) {
  const dim3 grid(xcd_grid(nqb, H, B));
  const bool split = nqb >= 4 && grid.x <= 768;
#define SPA_LAUNCH_F32(D, W) hipLaunchKernelGGL((attn_fwd_f32_kernel<D, W>), grid, dim3(64 * W), 0, st, args...)
  if (Dh == 32) {
    if (split) SPA_LAUNCH_F32(32, 4); else SPA_LAUNCH_F32(32, 1);
  } else {
    if (split) SPA_LAUNCH_F32(64, 4); else SPA_LAUNCH_F32(64, 1);
  }
#undef SPA_LAUNCH_F32
}
static int attention_common(const char* fn, const void* q, const void* k, const void* v,
                            int64_t q_stride, int64_t k_stride, int64_t v_stride, const int32_t* cu, const int32_t* key_lens, int B,
                            int n_max, int H, int Dh, int dtype, float softmax_scale, void* out,
                            float* lse, const Scatter& sc, void* stream, const float* v_scores = nullptr) {
  SPA_REQUIRE(q && k && v && (out || sc.y) && (cu || key_lens), SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(B >= 1 && n_max >= 1 && H >= 1, SPA_ERR_INVALID_ARG, "%s: B, max_seqlen, H must be >= 1", fn);
  SPA_REQUIRE((long)B * n_max < 2147483647L, SPA_ERR_INVALID_ARG, "%s: B*max_seqlen must be < 2^31", fn);
  SPA_REQUIRE(B <= 65535 && H <= 65535, SPA_ERR_INVALID_ARG, "%s: B and H must be <= 65535", fn);
  SPA_REQUIRE(((long)H * B + 8) * ((n_max + 31) / 32) < 2147483647L, SPA_ERR_INVALID_ARG,
              "%s: B*H*ceil(max_seqlen/32) must be < 2^31", fn);
  SPA_REQUIRE(dtype == SPA_F32 || dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: unknown dtype %d", fn, dtype);
  SPA_REQUIRE(Dh == 32 || Dh == 64, SPA_ERR_UNSUPPORTED, "%s: head dim %d not supported (32 or 64)", fn, Dh);
  const int64_t strides[3] = {q_stride, k_stride, v_stride};
  for (int64_t rs : strides) {
    SPA_REQUIRE(rs >= (int64_t)H * Dh, SPA_ERR_INVALID_ARG, "%s: row stride %ld < H*Dh", fn, (long)rs);
    // the kernels keep a lane's offset inside a tile (up to 128 rows) in 32 bits
    SPA_REQUIRE(rs < (1 << 24), SPA_ERR_INVALID_ARG, "%s: row stride %ld must be < 2^24 elements", fn, (long)rs);
    SPA_REQUIRE((rs * elem_size(dtype)) % 16 == 0, SPA_ERR_INVALID_ARG, "%s: row stride is not a multiple of 16 bytes", fn);
  }
  SPA_REQUIRE(aligned16(q) && aligned16(k) && aligned16(v) && aligned16(out), SPA_ERR_INVALID_ARG,
              "%s: q/k/v/out not 16-byte aligned", fn);
  SPA_REQUIRE(softmax_scale >= 0.f && std::isfinite(softmax_scale), SPA_ERR_INVALID_ARG,
              "%s: softmax_scale must be finite and >= 0 (0 = 1/sqrt(Dh))", fn);
  const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt((float)Dh);
  const long lse_stride = (long)B * n_max;
  hipStream_t st = as_stream(stream);
  if (dtype == SPA_F32) {
    SPA_REQUIRE(!group_open(), SPA_ERR_UNSUPPORTED, "%s: fp32 calls cannot be part of a group", fn);
    const int nqb = (n_max + 31) / 32;
    launch_f32(Dh, B, H, nqb, st, (const float*)q, (const float*)k, (const float*)v, (long)q_stride, (long)k_stride, (long)v_stride,
               cu, key_lens, n_max, H, scale, (float*)out, lse, lse_stride, sc, B, nqb);
  } else {
    const float scale_log2 = scale * 1.4426950408889634f;
    FwdArgs args = {(const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (long)q_stride, (long)k_stride, (long)v_stride, v_scores,
                    cu, key_lens, n_max, H, scale_log2, (__bf16*)out, lse, lse_stride, sc, B, 0, 0, 1};
    const bool d_after = sc.dvec != nullptr && !group_open() && !dy_apart(args, args, Dh);      // D in a launch of its own
    const int form = v_scores != nullptr ? (sc.dvec != nullptr && !d_after ? kFwdGatedD : kFwdGated) : sc.gathered ? kFwdGathered : kFwdPacked;
    const auto live = [&] { return key_lens == nullptr && live_tiles_apply(H, B); };
    // the tiled kernel's workgroups: of those resident together three a unit walk at head dim 32, two at 64, beside the fill
    const auto tiled_grid = [&] {
      args.nqb = (n_max + 127) / 128;
      const long all = xcd_grid(args.nqb, H, B);
      args.ntile = (int)(live() ? std::min<long>(all, (Dh == 32 ? 3 : 2) * 256) : all);
      const long rows = sc.y == nullptr ? 0 : sc.flat ? (long)sc.N : (long)B * sc.N;
      return (unsigned)(args.ntile + std::min<long>((rows + 31) / 32, 1024));
    };
    if (group_open()) {
      SPA_REQUIRE(Dh == 32 && key_lens == nullptr && (n_max > 256 || (form != kFwdGathered && B <= kWave)),
                  SPA_ERR_UNSUPPORTED,
                  "%s: this form cannot be part of a group", fn);
      if (n_max > 256) {
        const unsigned blocks = tiled_grid();
        return g_noted[form].add(fn, args, (blocks + 7) / 8 * 8);
      }
      args.nqb = (n_max + 31) / 32;
      args.waves = unit_waves(Dh, args.nqb, xcd_grid(args.nqb, H, B));
      return g_noted[form].add(fn, args, wave_groups(lpt64_grid(B, H, args.nqb), args.waves));
    }
#define SPA_LAUNCH(KERNEL, GRID, BLOCK, ARGS, ...)                                                            \
  do {                                                                                                        \
    if (sc.gathered) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFwdGathered>), GRID, BLOCK, 0, st, ARGS);       \
    else hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFwdPacked>), GRID, BLOCK, 0, st, ARGS);                     \
  } while (0)
#define SPA_LAUNCH_FORM(KERNEL, GRID, BLOCK, ARGS, ...)                                                       \
  do {                                                                                                        \
    if (form == kFwdGatedD) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFwdGatedD>), GRID, BLOCK, 0, st, ARGS);  \
    else if (form == kFwdGated) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFwdGated>), GRID, BLOCK, 0, st, ARGS); \
    else SPA_LAUNCH(KERNEL, GRID, BLOCK, ARGS, __VA_ARGS__);                                                  \
  } while (0)
#define SPA_ARGS                                                                                              \
  (const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (long)q_stride, (long)k_stride, (long)v_stride, cu,   \
      key_lens, n_max, H, scale_log2, (__bf16*)out, lse, lse_stride, sc
    // options attn_fwd_cfg (forces the tiled kernel with that launch shape), attn_fwd_short and
    // attn_fwd_wave_max select among the kernels below; unset, the measured best is taken
    const Options& opt = options();
    const bool tiled = opt.fwd_tiled;
    const bool use_whole = opt.fwd_whole;
    const int wave_max = opt.fwd_wave_max;
    if (!tiled && n_max <= wave_max && (!use_whole || is_gated(form))) {
      // short segments: one wave per (image, head, 32 queries)
      const int nqb = (n_max + 31) / 32;
      const dim3 grid(xcd_grid(nqb, H, B));
      args.nqb = nqb;
      // default: blocks dealt to the compute units by weight ("plain": numbered blindly)
      const bool step64 = opt.fwd_step64, plain = opt.fwd_plain;
      const int waves = step64 ? 1 : unit_waves(Dh, nqb, grid.x);
      const dim3 lgrid(lpt64_grid(B, H, nqb)), block(64 * waves);
#define SPA_WAVE(KERNEL, GRID, D)                                                       \
  do {                                                                                  \
    if (waves == 2) SPA_LAUNCH_FORM(KERNEL, GRID, block, args, 2, D, 32);          \
    else SPA_LAUNCH_FORM(KERNEL, GRID, block, args, 1, D, 32);                          \
  } while (0)
      if (step64) {
        if (Dh == 32) SPA_LAUNCH_FORM(attn_fwd_bf16_wave_kernel, grid, block, args, 1, 32, 64);
        else SPA_LAUNCH_FORM(attn_fwd_bf16_wave_kernel, grid, block, args, 1, 64, 64);
      } else if (!plain && B <= kWave) {
        if (Dh == 32) SPA_WAVE(attn_fwd_bf16_wave_lpt64_kernel, lgrid, 32);
        else SPA_WAVE(attn_fwd_bf16_wave_lpt64_kernel, lgrid, 64);
      } else {
        if (Dh == 32) SPA_WAVE(attn_fwd_bf16_wave_kernel, grid, 32);
        else SPA_WAVE(attn_fwd_bf16_wave_kernel, grid, 64);
      }
#undef SPA_WAVE
    } else if (!tiled && n_max <= 256 && !is_gated(form)) {
      // short segments: one workgroup per (image, head), whole segment in LDS
      const dim3 grid(H, B);
#define SPA_WHOLE(D)                                                                                          \
  do {                                                                                                        \
    if (n_max <= 64) SPA_LAUNCH(attn_fwd_bf16_whole_kernel, grid, dim3(128), SPA_ARGS, D, 64);       \
    else if (n_max <= 128) SPA_LAUNCH(attn_fwd_bf16_whole_kernel, grid, dim3(256), SPA_ARGS, D, 128); \
    else SPA_LAUNCH(attn_fwd_bf16_whole_kernel, grid, dim3(512), SPA_ARGS, D, 256);          \
  } while (0)
      if (Dh == 32) SPA_WHOLE(32); else SPA_WHOLE(64);
#undef SPA_WHOLE
    } else {
      const dim3 grid(tiled_grid());
      // All reads early take 165 registers at head dim 32, three workgroups a unit.  Up to as many blocks of capacity as these
      // slots hold; beyond, the fourth workgroup works for the launch itself or for another batch in flight.  us a step with 1 |
      // 2 | 4 streams, 8 heads of 32, late, then early: 1 x 4200 tokens, 5-40 % selected, 20.7 | 13.4 | 9.9 and 19.9 | 12.0 |
      // 9.1, 8 x 1024, 10-90 %, (512 blocks) 20.0 | 13.1 | 10.7 and 19.6 | 12.5 | 10.2, 8 x 1600 (832) 28.6 | 19.0 | 16.3
      // and 28.1 | 19.6 | 16.9, 16 x 1024 (1024) 23.2 | 16.2 | 14.0 and 22.9 | 17.2 | 14.8, 8 x 4200 (2112) 32.3 | 20.9 |
      // 19.1 and 31.7 | 22.2 | 20.6, 16 x 4200 51.6 | 41.5 | 39.6 and 52.7 | 43.7 | 41.2.
      // At head dim 64 some of the reads are early, as three workgroups a unit have registers for: late | some | all (two a
      // unit), 10-90 % selected: 23 x 391 tokens, 7 heads, 19.0 |
      // 18.0 | 18.5, 64 x 400, 12 heads, 46.9 | 46.3 | 54.1, 64 x 1024, 12 heads, 147 | 145 | 161, 32 x 4096, 6 heads, 393 | 393 | 391.
      const bool early = xcd_grid(args.nqb, H, B) <= 768;
      if (Dh == 64) SPA_LAUNCH_FORM(attn_fwd_bf16_tiled_kernel, grid, dim3(256), args, 64, 4, kReadSome);
      else if (early) SPA_LAUNCH_FORM(attn_fwd_bf16_tiled_kernel, grid, dim3(256), args, 32, 4, kReadAll);
      else SPA_LAUNCH_FORM(attn_fwd_bf16_tiled_kernel, grid, dim3(256), args, 32, 4, kReadLate);
    }
#undef SPA_ARGS
#undef SPA_LAUNCH
#undef SPA_LAUNCH_FORM
    if (d_after) launch_dvec_of(args, Dh, st);
  }
  return check_launch(fn);
}

}  // namespace spa

using namespace spa;

extern "C" int spa_packed_attention(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                    int64_t k_row_stride, int64_t v_row_stride, const int32_t* cu_seqlens, int B, int max_seqlen, int H, int Dh,
                                    int dtype, float softmax_scale, void* out, float* lse, void* stream) {
  SPA_REQUIRE(cu_seqlens, SPA_ERR_INVALID_ARG, "spa_packed_attention: cu_seqlens is null");
  SPA_REQUIRE(out, SPA_ERR_INVALID_ARG, "spa_packed_attention: out is null");
  const Scatter none = {nullptr, nullptr, nullptr, nullptr, 0, 0, 0, nullptr};
  return attention_common("spa_packed_attention", q, k, v, q_row_stride, k_row_stride, v_row_stride, cu_seqlens, nullptr, B, max_seqlen,
                          H, Dh, dtype, softmax_scale, out, lse, none, stream);
}

extern "C" int spa_packed_attention_running_max(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                                int64_t k_row_stride, int64_t v_row_stride, const int32_t* cu_seqlens, int B,
                                                int max_seqlen, int H, int Dh, int dtype, float softmax_scale, void* out,
                                                float* lse, void* stream) {
  return spa_packed_attention(q, k, v, q_row_stride, k_row_stride, v_row_stride, cu_seqlens, B, max_seqlen, H, Dh, dtype,
                              softmax_scale, out, lse, stream);
}

extern "C" int spa_padded_attention(const void* q, const void* k, const void* v, int64_t row_stride,
                                    const int32_t* seqlens, int B, int n_pad, int H, int Dh, int dtype,
                                    float softmax_scale, void* out, void* stream) {
  SPA_REQUIRE(seqlens, SPA_ERR_INVALID_ARG, "spa_padded_attention: seqlens is null");
  SPA_REQUIRE(out, SPA_ERR_INVALID_ARG, "spa_padded_attention: out is null");
  const Scatter none = {nullptr, nullptr, nullptr, nullptr, 0, 0, 0, nullptr};
  return attention_common("spa_padded_attention", q, k, v, row_stride, row_stride, row_stride, nullptr, seqlens, B, n_pad, H, Dh,
                          dtype, softmax_scale, out, nullptr, none, stream);
}

extern "C" int spa_packed_attention_unpack(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                           int64_t k_row_stride, int64_t v_row_stride,
                                           const int32_t* cu_seqlens, const int32_t* gather_idx,
                                           const int32_t* inv_pos, const void* base, int B, int N, int H, int Dh,
                                           int dtype, float softmax_scale, void* out, float* lse, void* y,
                                           void* stream) {
  SPA_REQUIRE(cu_seqlens && gather_idx && inv_pos && y, SPA_ERR_INVALID_ARG,
              "spa_packed_attention_unpack: null pointer");
  SPA_REQUIRE(aligned16(y) && aligned16(base), SPA_ERR_INVALID_ARG,
              "spa_packed_attention_unpack: y / base not 16-byte aligned");
  const Scatter sc = {gather_idx, inv_pos, base, y, N, 0, 0, nullptr};
  return attention_common("spa_packed_attention_unpack", q, k, v, q_row_stride, k_row_stride, v_row_stride,
                          cu_seqlens, nullptr, B, N, H, Dh, dtype, softmax_scale, out, lse, sc, stream);
}

extern "C" int spa_gathered_attention_unpack(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                             int64_t k_row_stride, int64_t v_row_stride,
                                             const int32_t* cu_seqlens, const int32_t* gather_idx,
                                             const int32_t* inv_pos, const void* base, int B, int N, int H, int Dh,
                                             int dtype, float softmax_scale, void* out, float* lse, void* y,
                                             void* stream) {
  const char* fn = "spa_gathered_attention_unpack";
  SPA_REQUIRE(cu_seqlens && gather_idx && inv_pos && y, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(aligned16(y) && aligned16(base), SPA_ERR_INVALID_ARG, "%s: y / base not 16-byte aligned", fn);
  const Scatter sc = {gather_idx, inv_pos, base, y, N, 0, 1, nullptr};
  return attention_common(fn, q, k, v, q_row_stride, k_row_stride, v_row_stride, cu_seqlens, nullptr, B, N, H, Dh,
                          dtype, softmax_scale, out, lse, sc, stream);
}

static int gated_attention_unpack(const char* fn, const void* q, const void* k, const void* x, int64_t q_row_stride,
                                  int64_t k_row_stride, int64_t x_row_stride, const float* scores, const int32_t* cu_seqlens,
                                  const int32_t* gather_idx, const int32_t* inv_pos, const void* base, int B, int N, int H,
                                  int Dh, int dtype, float softmax_scale, void* out, float* lse, void* y, const void* dy,
                                  float* dvec, void* stream) {
  SPA_REQUIRE(scores && cu_seqlens && gather_idx && inv_pos && y, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(aligned16(y) && aligned16(base) && aligned16(dy), SPA_ERR_INVALID_ARG, "%s: y / base / dy not 16-byte aligned", fn);
  SPA_REQUIRE(dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: bf16 only (use spa_pack_pair + spa_packed_attention_unpack)", fn);
  const Scatter sc = {gather_idx, inv_pos, base, y, N, 0, 1, nullptr, static_cast<const __bf16*>(dy), dvec};
  return attention_common(fn, q, k, x, q_row_stride, k_row_stride, x_row_stride, cu_seqlens, nullptr, B, N, H, Dh, dtype,
                          softmax_scale, out, lse, sc, stream, scores);
}

extern "C" int spa_gated_attention_unpack(const void* q, const void* k, const void* x, int64_t q_row_stride,
                                          int64_t k_row_stride, int64_t x_row_stride, const float* scores,
                                          const int32_t* cu_seqlens, const int32_t* gather_idx, const int32_t* inv_pos,
                                          const void* base, int B, int N, int H, int Dh, int dtype, float softmax_scale,
                                          void* out, float* lse, void* y, void* stream) {
  return gated_attention_unpack("spa_gated_attention_unpack", q, k, x, q_row_stride, k_row_stride, x_row_stride, scores,
                                cu_seqlens, gather_idx, inv_pos, base, B, N, H, Dh, dtype, softmax_scale, out, lse, y, nullptr,
                                nullptr, stream);
}

extern "C" int spa_gated_attention_unpack_dvec(const void* q, const void* k, const void* x, int64_t q_row_stride,
                                               int64_t k_row_stride, int64_t x_row_stride, const float* scores,
                                               const int32_t* cu_seqlens, const int32_t* gather_idx, const int32_t* inv_pos,
                                               const void* base, int B, int N, int H, int Dh, int dtype, float softmax_scale,
                                               void* out, float* lse, void* y, const void* dy, void* workspace,
                                               size_t workspace_bytes, void* stream) {
  const char* fn = "spa_gated_attention_unpack_dvec";
  SPA_REQUIRE(dy && out && lse, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(workspace != nullptr && workspace_bytes >= spa_attention_bwd_workspace_bytes(B, N, H, Dh, dtype), SPA_ERR_WORKSPACE,
              "%s: the workspace of the backward is needed, %zu bytes given", fn, workspace_bytes);
  return gated_attention_unpack(fn, q, k, x, q_row_stride, k_row_stride, x_row_stride, scores, cu_seqlens, gather_idx, inv_pos,
                                base, B, N, H, Dh, dtype, softmax_scale, out, lse, y, dy, static_cast<float*>(workspace), stream);
}

extern "C" int spa_selected_attention_unpack(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                             int64_t k_row_stride, int64_t v_row_stride, const uint8_t* mask,
                                             const void* base, int B, int N, int H, int Dh, int dtype,
                                             float softmax_scale, void* y, void* stream) {
  const char* fn = "spa_selected_attention_unpack";
  SPA_REQUIRE(q && k && v && mask && y, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(B >= 1 && N >= 1 && H >= 1, SPA_ERR_INVALID_ARG, "%s: B, N, H must be >= 1", fn);
  SPA_REQUIRE(dtype == SPA_F32 || dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: unknown dtype %d", fn, dtype);
  SPA_REQUIRE(N <= 256, SPA_ERR_UNSUPPORTED, "%s: N = %d > 256 tokens per image (use index-only spa_pack + spa_gathered_attention_unpack)", fn, N);
  SPA_REQUIRE(Dh == 32 || Dh == 64, SPA_ERR_UNSUPPORTED, "%s: head dim %d not supported (32 or 64)", fn, Dh);
  SPA_REQUIRE(B <= 65535 && H <= 65535 && (long)B * N < 2147483647L, SPA_ERR_INVALID_ARG, "%s: B, H <= 65535 and B*N < 2^31", fn);
  SPA_REQUIRE(((long)H * B + 8) * ((N + 31) / 32) < 2147483647L, SPA_ERR_INVALID_ARG, "%s: B*H*ceil(N/32) must be < 2^31", fn);
  const int64_t strides[3] = {q_row_stride, k_row_stride, v_row_stride};
  for (int64_t rs : strides) {
    SPA_REQUIRE(rs >= (int64_t)H * Dh && rs < (1 << 24), SPA_ERR_INVALID_ARG, "%s: row stride %ld outside [H*Dh, 2^24)", fn, (long)rs);
    SPA_REQUIRE((rs * elem_size(dtype)) % 16 == 0, SPA_ERR_INVALID_ARG, "%s: row stride is not a multiple of 16 bytes", fn);
  }
  SPA_REQUIRE(aligned16(q) && aligned16(k) && aligned16(v) && aligned16(y) && aligned16(base), SPA_ERR_INVALID_ARG,
              "%s: q / k / v / y / base not 16-byte aligned", fn);
  SPA_REQUIRE(softmax_scale >= 0.f && std::isfinite(softmax_scale), SPA_ERR_INVALID_ARG,
              "%s: softmax_scale must be finite and >= 0 (0 = 1/sqrt(Dh))", fn);
  const float scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt((float)Dh);
  const float scale_log2 = scale * 1.4426950408889634f;
  const Scatter sc = {nullptr, nullptr, base, y, N, 0, 1, mask};
  const int nqb = (N + 31) / 32;
  const dim3 grid(xcd_grid(nqb, H, B));
  if (dtype == SPA_F32) {
    SPA_REQUIRE(!group_open(), SPA_ERR_UNSUPPORTED, "%s: fp32 calls cannot be part of a group", fn);
    launch_f32(Dh, B, H, nqb, as_stream(stream), (const float*)q, (const float*)k, (const float*)v, (long)q_row_stride,
               (long)k_row_stride, (long)v_row_stride, (const int32_t*)nullptr, (const int32_t*)nullptr, N, H, scale, (float*)nullptr,
               (float*)nullptr, 0L, sc, B, nqb);
    return check_launch(fn);
  }
  FwdArgs args = {(const __bf16*)q, (const __bf16*)k, (const __bf16*)v, (long)q_row_stride, (long)k_row_stride,
                        (long)v_row_stride, nullptr, nullptr, nullptr, N, H, scale_log2, nullptr, nullptr, 0L, sc, B, nqb, 0, 1};
  if (group_open()) {
    SPA_REQUIRE(Dh == 32, SPA_ERR_UNSUPPORTED, "%s: this form cannot be part of a group", fn);
    args.waves = unit_waves(Dh, nqb, grid.x);
    return g_noted[1].add(fn, args, wave_groups(grid.x, args.waves));
  }
  const int waves = unit_waves(Dh, nqb, grid.x);
#define SPA_MASK(D, W) hipLaunchKernelGGL((attn_fwd_bf16_wave_mask_kernel<D, 32, W>), grid, dim3(64 * W), 0, as_stream(stream), args)
#define SPA_MASK_WAVES(D)                 \
  do {                                    \
    if (waves == 2) SPA_MASK(D, 2);  \
    else SPA_MASK(D, 1);                  \
  } while (0)
  if (Dh == 32) SPA_MASK_WAVES(32); else SPA_MASK_WAVES(64);
#undef SPA_MASK
#undef SPA_MASK_WAVES
  return check_launch(fn);
}

extern "C" int spa_segment_attention_unpack(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                            int64_t k_row_stride, int64_t v_row_stride,
                                            const int32_t* seg_cu_seqlens, int n_segments, int max_seqlen,
                                            const int32_t* gather_idx, const int32_t* inv_pos, const void* base,
                                            int64_t rows, int H, int Dh, int dtype, float softmax_scale,
                                            void* out, float* lse, void* y, void* stream) {
  const char* fn = "spa_segment_attention_unpack";
  SPA_REQUIRE(seg_cu_seqlens && gather_idx && inv_pos && y, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(rows >= 1 && rows < 2147483647L, SPA_ERR_INVALID_ARG, "%s: rows must be in [1, 2^31)", fn);
  SPA_REQUIRE(aligned16(y) && aligned16(base), SPA_ERR_INVALID_ARG, "%s: y / base not 16-byte aligned", fn);
  const Scatter sc = {gather_idx, inv_pos, base, y, (int)rows, 1, 0, nullptr};
  return attention_common(fn, q, k, v, q_row_stride, k_row_stride, v_row_stride, seg_cu_seqlens, nullptr, n_segments,
                          max_seqlen, H, Dh, dtype, softmax_scale, out, lse, sc, stream);
}

extern "C" int spa_gathered_segment_attention_unpack(const void* q, const void* k, const void* v, int64_t q_row_stride,
                                                     int64_t k_row_stride, int64_t v_row_stride,
                                                     const int32_t* seg_cu_seqlens, int n_segments, int max_seqlen,
                                                     const int32_t* gather_idx, const int32_t* inv_pos, const void* base,
                                                     int64_t rows, int H, int Dh, int dtype, float softmax_scale, void* out,
                                                     float* lse, void* y, void* stream) {
  const char* fn = "spa_gathered_segment_attention_unpack";
  SPA_REQUIRE(seg_cu_seqlens && gather_idx && inv_pos && y, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(rows >= 1 && rows < 2147483647L, SPA_ERR_INVALID_ARG, "%s: rows must be in [1, 2^31)", fn);
  SPA_REQUIRE(aligned16(y) && aligned16(base), SPA_ERR_INVALID_ARG, "%s: y / base not 16-byte aligned", fn);
  const Scatter sc = {gather_idx, inv_pos, base, y, (int)rows, 1, 1, nullptr};
  return attention_common(fn, q, k, v, q_row_stride, k_row_stride, v_row_stride, seg_cu_seqlens, nullptr, n_segments,
                          max_seqlen, H, Dh, dtype, softmax_scale, out, lse, sc, stream);
}
