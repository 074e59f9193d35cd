// The main loop shared by the projection GEMMs (bf16 MFMA, fp32 accumulation): operand tiles go from
// memory straight to LDS (global_load_lds, 16 bytes a lane) through a ring of two to four buffers, so the
// loads of the next tiles are in flight without a register, a store or a wait for each other; the only
// waits are one counted vmcnt and one barrier per 64-deep contraction step.  The barrier stands before the last
// products of the step before it, whose operands are in registers by then: they cover the first LDS reads of the
// step, and all buffers can be filled before the first.
//
// What bounds it: 256 x 256, called again and again on all units, a step takes 1.65 us with random operands and 1.14 with
// zeros (the products alone .93 with either, the loads alone .86, the reads alone .7 | .42 for rows | deep operands): the
// clock falls with the power that the operands' bits cost, and at 1.65 us the products run at 1.3 PFLOP/s.  A wave
// issues an LDS read in 15 to 17 cycles, a matrix instruction takes 32: a wave's reads stand between its products, not in
// front of them (rows of 768 -> 2304, 12544 of them, 49.6 -> 46.5 us with that and the pieces' order below).
//
// A direct load puts a wave's 64 pieces of 16 bytes next to each other, so rows cannot be padded;
// instead the pieces of a row are permuted on the way in (each lane chooses which piece it fetches) and
// un-permuted in the fragment reads:
//   rows operand ([rows][64], contraction along the row):  piece c of row r sits at c ^ MF::turn(r)
//   deep operand ([64][cols], contraction down the rows):  piece c of row r sits at c ^ 4 (r & 3)
// which spreads the 16-byte reads of the rows that are read together, and the transposing reads of 4 rows, over all
// banks: 4.2 cycles for a 16-byte read and 2.2 for a transposing one with eight waves reading (r & 7 for the 32-row
// fragments, of whose rows r and r + 8 meet: 8.0; 256 x 256 tiles 3 % slower).
#pragma once

#include <type_traits>

#include "attn_tiles.h"
#include "spa_common.h"

namespace spa {

constexpr int kGaK = 64;             // contraction step

// 16 bytes of zeros for every lane whose piece lies outside the operand
static __device__ __align__(256) const uint32_t gemm_zeros[64] = {};

// 16 bytes per lane from src to the wave's 1 KB at LDS byte address dst (lane l at dst + 16 l; M0 holds
// dst, which the load may use one wait state after it is written).  Inline assembly because the compiler
// takes the builtin's load for one that may return through either counter and from then on waits for
// lgkmcnt(0) before every use of an LDS read; what is in flight is counted by the waits below, and by
// the compiler's own waits on the safe side.
__device__ __forceinline__ void load_to_lds(const __bf16* src, uint32_t dst) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_memory() {    // at most N vector memory operations still in flight, and no LDS read
  static_assert(N >= 0 && N < 64, "vmcnt has six bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x070);
}

// The matrix instruction of a tile: EDGE x EDGE products of DEPTH contraction elements.  Lane l holds row (or
// column) l % EDGE and elements 8 (l / EDGE) .. + 7 of an operand; of a product, column l % EDGE and, in group g,
// rows row(g, l) .. + 3.
struct Mfma32 {
  static constexpr int kEdge = 32, kDepth = 16, kGroups = 4;
  typedef floatx16 Acc;
  __device__ static __forceinline__ Acc mul(bf16x8 a, bf16x8 b, Acc c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
  __device__ static __forceinline__ int row(int g, int lane) { return 8 * g + 4 * (lane >> 5); }
  __device__ static __forceinline__ int turn(int r) { return r >> 1 & 7; }     // of a rows operand's pieces
};
struct Mfma16 {
  static constexpr int kEdge = 16, kDepth = 32, kGroups = 1;
  typedef floatx4 Acc;
  __device__ static __forceinline__ Acc mul(bf16x8 a, bf16x8 b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
  __device__ static __forceinline__ int row(int, int lane) { return 4 * (lane >> 4); }
  __device__ static __forceinline__ int turn(int r) { return r & 7; }
};

// Operand with the contraction along its rows: fragment of rows r0 .. + EDGE - 1, contraction DEPTH kk .. + DEPTH - 1.
template <class MF>
__device__ __forceinline__ bf16x8 rows_frag(const __bf16* tile, int r0, int kk, int lane) {
  const int r = r0 + lane % MF::kEdge;
  return *reinterpret_cast<const bf16x8*>(tile + r * kGaK + (((MF::kDepth / 8 * kk + lane / MF::kEdge) ^ MF::turn(r)) << 3));
}
// Operand with the contraction down its rows (COLS columns): fragment of columns c0 .. c0+31, contraction
// rows 16 kk .. + 15, by the transposing read: within each block of 16 lanes lane i, element e, receives
// what lane (4 e + i / 4) of the block addressed at its own element i % 4.
template <int COLS>
__device__ __forceinline__ bf16x8 deep_frag(const __bf16* tile, int kk, int c0, int lane) {
  const int blk = lane >> 4, s = lane & 15;
  const int row = 16 * kk + 8 * (blk >> 1) + (s >> 2);
  const int piece = ((c0 >> 3) ^ (4 * (s >> 2))) + 2 * (blk & 1) + ((s & 3) >> 1);
  const __bf16* p = tile + row * COLS + piece * 8 + 4 * (s & 1);
  typedef shortx4_lds __attribute__((address_space(3))) * lds_ptr;
  const shortx4_lds lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
  const shortx4_lds hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * COLS));
  const bf16x4 l4 = __builtin_bit_cast(bf16x4, lo), h4 = __builtin_bit_cast(bf16x4, hi);
  return __builtin_shufflevector(l4, h4, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Deep operand in blocks of 64 columns ([columns / 64][64][64]): fragment of columns c0 .. c0+15, contraction rows
// 32 kk .. + 31.  Piece c of row r sits at c ^ (2 (r / 2 % 2) + 4 (r / 8 % 2)): the 8 rows that 32 lanes read
// together fall on distinct banks.
__device__ __forceinline__ bf16x8 deep_block_frag(const __bf16* tile, int kk, int c0, int lane) {
  const int blk = lane >> 4, s = lane & 15, row = 32 * kk + 8 * blk + (s >> 2);
  const int piece = (((c0 & 63) >> 3) + ((s & 3) >> 1)) ^ (2 * (s >> 3) + 4 * (blk & 1));
  const __bf16* p = tile + (c0 >> 6) * (64 * kGaK) + row * 64 + piece * 8 + 4 * (s & 1);
  typedef shortx4_lds __attribute__((address_space(3))) * lds_ptr;
  const shortx4_lds lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
  const shortx4_lds hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * 64));
  const bf16x4 l4 = __builtin_bit_cast(bf16x4, lo), h4 = __builtin_bit_cast(bf16x4, hi);
  return __builtin_shufflevector(l4, h4, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Which piece a thread fetches: piece `col` (elements) of tile row `row` for u = 0 .. count - 1.
template <class MF, int ROWS, int THREADS>
struct RowsPieces {
  static constexpr int kCount = ROWS * 8 / THREADS, kRowStep = THREADS / 8;
  static_assert(kRowStep % 16 == 0, "a thread keeps its permuted column");
  __device__ static __forceinline__ int row(int tid, int u) { return (tid >> 3) + u * kRowStep; }
  __device__ static __forceinline__ int col(int tid, int) { return ((tid & 7) ^ MF::turn(tid >> 3)) * 8; }
};
template <int COLS, int THREADS, int DEPTH = kGaK>
struct DeepPieces {
  static constexpr int kPerRow = COLS / 8, kCount = DEPTH * kPerRow / THREADS, kRowStep = THREADS / kPerRow;
  static_assert(kRowStep % 4 == 0, "a thread keeps its permuted column");
  __device__ static __forceinline__ int row(int tid, int u) { return tid / kPerRow + u * kRowStep; }
  __device__ static __forceinline__ int col(int tid, int) {
    return ((tid % kPerRow) ^ (4 * ((tid / kPerRow) & 3))) * 8;
  }
};
template <int COLS, int THREADS>
struct DeepBlocks {                  // one block of 64 columns a step of u: a thread keeps its row
  static constexpr int kCount = COLS / 64;
  static_assert(THREADS == kGaK * 8, "a piece a thread and block");
  __device__ static __forceinline__ int row(int tid, int) { return tid >> 3; }
  __device__ static __forceinline__ int col(int tid, int u) {
    const int r = tid >> 3;
    return u * 64 + ((tid & 7) ^ (2 * (r >> 1 & 1) + 4 * (r >> 3 & 1))) * 8;
  }
};

// acc[i][j] += sum over nk contraction steps of DEPTH of (B fragment j) x (A fragment i): MFMA tiles whose
// rows are B's index and whose columns are A's.  The wave's block is TM * 32 of A by TN * 32 of B.
// next_a(u, t, inside) / next_b(u, t, inside): address of the thread's u-th piece of step t (called for t = 0, 1, ... in
// order, so they may step a pointer; inside: t + 1 < nk).  frag_a(tile, i, kk), frag_b(tile, j, kk): fragments;
// beside(af): called with the A fragments of every 16 contraction elements; stepped(t): when acc holds steps 0 .. t, of all but the
// last; last(): before the last barrier.  All threads
// call it.  On return nothing is in flight and every wave is past its last read of the buffers.  SA, SB: steps of A and B in LDS; A may have
// one more (rows that nobody has fetched yet take longer to come than the other operand, which all units share).
struct Nothing {
  template <class T> __device__ __forceinline__ void operator()(const T&) const {}
};
template <class MF, int A_ELEMS, int B_ELEMS, int NA, int NB, int SA, int SB, int THREADS, int TM, int TN, int DEPTH = kGaK, class FA,
          class FB, class RA, class RB, class LS, class BS = Nothing, class ST = Nothing>
__device__ __forceinline__ void gemm_async_loop(__bf16* lds, int nk, FA&& next_a, FB&& next_b, RA&& frag_a, RB&& frag_b,
                                                typename MF::Acc (&acc)[TM][TN], LS&& last, BS&& beside = BS{},
                                                ST&& stepped = ST{}) {
  constexpr int KK = DEPTH / MF::kDepth, LOADS = NA + NB;
  static_assert(KK % 2 == 0, "the fragments of neighbouring groups take turns");
  static_assert(SB >= 2 && (SA == SB || SA == SB + 1), "waits by whole groups of loads");
  // Place of a group's fragment reads and loads among its products: RP fragments after each product from the first on,
  // then a load after each.  With two buffers and one wave a SIMD, or two of workgroups that are not in step, the loads of a
  // step go first (dealt out: 2304 -> 768, 1568 rows, 26 -> 32 us).
  constexpr int P = TM * TN, R = TM + TN, RP = (2 * R + P - 1) / P, READS = (R + RP - 1) / RP;
  constexpr bool kLoadsFirst = THREADS == 256;
  constexpr int PER_GROUP = P - READS;
  static_assert(READS < P && (kLoadsFirst || LOADS <= KK * PER_GROUP), "every read and every load has its place");
  // one ring of A and B together, or one of A and one of B behind it
  constexpr bool kOneRing = SA == SB;
  constexpr int A_STEP = kOneRing ? A_ELEMS + B_ELEMS : A_ELEMS, B_STEP = kOneRing ? A_STEP : B_ELEMS;
  static_assert(kOneRing || !kLoadsFirst, "one ring where the loads go first");
  constexpr int B_FIRST = kOneRing ? A_ELEMS : SA * A_ELEMS;
  const uint32_t dst_a = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds +
                         __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 1024;
  // load q of step t, A's before B's in one ring; in two B's first, they are waited for first
  auto issue_a = [&](int q, int t, int buf, auto inside) { load_to_lds(next_a(q, t, inside), dst_a + buf * (A_STEP * 2) + q * (THREADS * 16)); };
  auto issue_b = [&](int q, int t, int buf, auto inside) {
    load_to_lds(next_b(q, t, inside), dst_a + B_FIRST * 2 + buf * (B_STEP * 2) + q * (THREADS * 16));
  };
#pragma unroll
  for (int s = 0; s < SA; ++s)
    if (s < nk) {
#pragma unroll
      for (int q = 0; q < (kOneRing ? NA : 0); ++q) issue_a(q, s, s, std::false_type{});
#pragma unroll
      for (int q = 0; q < (s < SB ? NB : 0); ++q) issue_b(q, s, s, std::false_type{});
#pragma unroll
      for (int q = 0; q < (kOneRing ? 0 : NA); ++q) issue_a(q, s, s, std::false_type{});
    }
  bf16x8 af[2][TM], bfr[2][TN];
  const __bf16 *a = lds, *b = lds + B_FIRST;
  auto read = [&](int kk, int r) {                   // fragment r of group kk: a and b in turn while both last
    const int both = 2 * (TM < TN ? TM : TN);
    const bool is_a = r < both ? r % 2 == 0 : TM > TN;
    const int i = r < both ? r / 2 : r - both / 2;
    if (is_a) af[kk & 1][i] = frag_a(a, i, kk);
    else bfr[kk & 1][i] = frag_b(b, i, kk);
  };
  int buf_a = 0, buf_b = 0, freed_a = 0, freed_b = 0;      // buffers of this step and of the one before it
  bool more_a = false, more_b = false;                     // the loads that fill the freed buffers exist
  // load q of those that follow step t: A of step t + SA, B of step t + SB.  inside: all of them exist and none is of the last
  // step, which may be partial: no test and no branch
  auto issue = [&](int q, int t, auto inside) {
    if constexpr (kOneRing) {
      if (inside || more_a) q < NA ? issue_a(q, t + SA, freed_a, inside) : issue_b(q - NA, t + SB, freed_a, inside);
    } else if (q < NB) {
      if (inside || more_b) issue_b(q, t + SB, freed_b, inside);
    } else if (inside || more_a) {
      issue_a(q - NB, t + SA, freed_a, inside);
    }
  };
  // the products of group kk beside the reads of group `next` and the loads that follow step t from number `from` on
  auto group = [&](int kk, int next, bool loads, int from, int t, auto inside) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int n = i * TN + j;
        acc[i][j] = MF::mul(bfr[kk & 1][j], af[kk & 1][i], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        if (n < READS) {
#pragma unroll
          for (int r = n * RP; r < (n + 1) * RP && r < R; ++r) read(next, r);
        } else if (!kLoadsFirst && from + n - READS < LOADS) {
          if (loads) issue(from + n - READS, t, inside);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    beside(af[kk & 1]);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto step = [&](int t, auto inside) {
#pragma unroll
    for (int kk = 0; kk + 1 < KK; ++kk) group(kk, kk + 1, true, (kk + 1) * PER_GROUP, t - 1, inside);
    // this wave's pieces of step t + 1 have arrived (near the end fewer younger ones are in flight), and its
    // reads of step t
    if (SA > 2 && !inside && t + SA - 1 >= nk) wait_memory<0>();
    else wait_memory<(SB - 2) * LOADS + (SA - SB) * NA>();
    __builtin_amdgcn_s_barrier();                   // and everybody's
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    freed_a = buf_a;
    freed_b = buf_b;
    buf_a = buf_a + 1 == SA ? 0 : buf_a + 1;
    buf_b = buf_b + 1 == SB ? 0 : buf_b + 1;
    a = lds + buf_a * A_STEP;
    b = kOneRing ? a + B_FIRST : lds + B_FIRST + buf_b * B_STEP;
    more_a = inside || t + SA < nk;
    more_b = inside || t + SB < nk;
    if (kLoadsFirst && more_a) {
#pragma unroll
      for (int q = 0; q < LOADS; ++q) issue(q, t, inside);
    }
    group(KK - 1, 0, true, 0, t, inside);
    stepped(t);
  };
  if (nk > 0) {
    if (SA <= nk) wait_memory<(SB - 1) * LOADS + (SA - SB) * NA>();
    else wait_memory<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < R; ++r) read(0, r);
    __builtin_amdgcn_sched_barrier(0);
  }
  int t = 0;
  if (nk > 1) step(t++, std::false_type{});
  for (; t + SA + 1 < nk; ++t) step(t, std::true_type{});
  for (; t + 1 < nk; ++t) step(t, std::false_type{});
  if (nk > 0) {
#pragma unroll
    for (int kk = 0; kk + 1 < KK; ++kk) group(kk, kk + 1, false, 0, 0, std::false_type{});
  }
  last();
  __syncthreads();
  if (nk > 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = MF::mul(bfr[1][j], af[1][i], acc[i][j]);
    beside(af[1]);
  }
}

}  // namespace spa
