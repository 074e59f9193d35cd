// Gate scoring + hard selection (Section 3.2, equations for s and r_p), the 2x2 max-pool
// that resizes up-scale scores, and the gate backward with the selection loss
// (Section 3.3).  All kernels are bandwidth-bound: every feature row is read once with
// 16-byte loads, a group of G lanes per token, fp32 accumulation.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "group.h"
#include "spa_common.h"

namespace spa {

constexpr int kGateThreads = 256;
constexpr int kMaxGateC = 8192;

template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int kElems = 4;
  // dx is the last thing the backward pass writes and nothing here reads it again: non-temporal
  __device__ static __forceinline__ void store(float* p, const float (&f)[4]) {
    floatx4 v = {f[0], f[1], f[2], f[3]};
    __builtin_nontemporal_store(v, reinterpret_cast<floatx4*>(p));
  }
};
template <> struct Vec16<__bf16> {
  static constexpr int kElems = 8;
  __device__ static __forceinline__ void store(__bf16* p, const float (&f)[8]) {
    floatx8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = f[i];
    __builtin_nontemporal_store(float_to_bf16x8(v), reinterpret_cast<bf16x8*>(p));
  }
};

template <typename T> struct Raw16;
template <> struct Raw16<float> { using type = floatx4; };
template <> struct Raw16<__bf16> { using type = bf16x8; };
__device__ __forceinline__ void widen(floatx4 v, float (&f)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = v[i];
}
__device__ __forceinline__ void widen(bf16x8 v, float (&f)[8]) {
  const floatx8 w = bf16x8_to_float(v);
#pragma unroll
  for (int i = 0; i < 8; ++i) f[i] = w[i];
}

// Sum over groups of G neighbouring lanes, in every lane, in the order of exchanges with lane ^ G/2, ^ G/4, ... ^ 1, in the
// vector ALU: the two halves and the two 16-lane rows of a half by the lane swaps, ^ 8 as a rotation of the row by 8, ^ 4 as
// one by 4 once both halves of a row hold the same (groups of 8: as two shifts), ^ 2 and ^ 1 inside a quad.  An
// exchange through LDS takes 85 cycles, one of these 8 to 16, and the dot products wait for each of them.
__device__ __forceinline__ float add_lane_xor32(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const unsigned a = r[0], b = r[1];
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
__device__ __forceinline__ float add_lane_xor16(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned a = r[0], b = r[1];
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
template <int G>
__device__ __forceinline__ float group_sum(float v) {
  constexpr int kRor = 0x120;
  if (G > 32) v = add_lane_xor32(v);
  if (G > 16) v = add_lane_xor16(v);
  if (G > 8) v += dpp_move<kRor + 8>(v);
  if (G > 8) v += dpp_move<kRor + 4>(v);
  else v += lane_xor<4>(v);
  v += lane_xor<2>(v);
  return v + lane_xor<1>(v);
}

// Lanes per token: by the row's 16-byte chunks (the same for every launch of the gate)
__host__ __device__ constexpr int gate_lanes(int chunks) { return chunks <= 8 ? 8 : chunks <= 64 ? 16 : chunks <= 256 ? 32 : 64; }
// The order of a token's sum.  The gate backward forms the sum again to see which side won the maximum with the
// up-scale score, on up to 64 lanes where the forward has 16 or 32, and near a tie the last bit decides: a lane of the
// forward therefore keeps gate_chains(G) partial sums, chunk number k of the lane in chain k % gate_chains(G), and
// folds them as the wider exchange of the backward does (lane ^ 32, then lane ^ 16).  Both then agree bit for bit.
__host__ __device__ constexpr int gate_chains(int G) { return G == 16 ? 4 : G == 32 ? 2 : 1; }
template <int A>
__device__ __forceinline__ float fold_chains(const float (&acc)[A]) {
  if constexpr (A == 4) return (acc[0] + acc[2]) + (acc[1] + acc[3]);
  else if constexpr (A == 2) return acc[0] + acc[1];
  else return acc[0];
}

// One group of G lanes per token; the group strides over the row's 16-byte chunks.
// kPool: s_up is the score map of the finer stage, [B, 2 gh, 2 gw], and is 2x2 max-pooled on
// the fly (Section 3.2: up-scale scores adjusted via max-pooling); the pooled value is also
// written to s_up_pooled when that is given (the backward pass needs it).
struct PoolGrid {
  int gh, gw;            // this stage's grid, N = gh * gw
  float* s_up_pooled;    // [B, N] or null
};

// Packing index built by the gate launch itself (Section 3.2 "Token Packing" needs nothing but the
// selection): the workgroup that finishes LAST (one arrival counter, no waiting anywhere) walks
// the mask once and writes cu_seqlens, gather_idx, inv_pos, total (and counts), exactly what
// spa_pack writes.  arrive == nullptr: off.
struct IndexOut {
  int32_t* cu_seqlens;   // [B+1]
  int32_t* gather_idx;   // [B*N]
  int32_t* inv_pos;      // [B*N]
  int32_t* total;        // [1] or null
  int32_t* counts;       // [B] or null
  unsigned* arrive;      // kArriveWords words, zero before the launch, zero again after it
};
// Arrival is counted in two levels, 16 group counters and a root: atomics on ONE address are served
// one after the other (about 25 ns each here, 50 us for the 2100 workgroups of a 33600-token
// batch), and so are atomics on neighbouring lines (they meet in one memory channel), so the
// counters lie 4352 bytes apart.
constexpr int kArriveGroups = 16, kArriveStride = 1088;             // words between counters (4352 bytes)
constexpr int kArriveWords = (kArriveGroups + 1) * kArriveStride;

// number of non-zero bytes in a 32-bit word
__device__ __forceinline__ int nonzero_bytes_u32(uint32_t w) {
  const uint32_t t = (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;
  return __popc(t);
}

// One workgroup of kGateThreads threads: stable compaction index of mask[0 .. ntok) (tokens of image b
// are [b*N, (b+1)*N)).  In a round, thread t owns the 16 consecutive tokens [4096 r + 16 t, + 16)
// (consecutive threads, consecutive groups: the index stores of a wave are contiguous); the
// mask words of up to kRounds rounds are fetched first, as independent 32-bit agent-scope loads (the
// mask is 16-byte aligned; other XCDs wrote these bytes in this same launch), so 32768 tokens cost
// one trip to memory, then every round is one scan over the workgroup and a walk of 16 tokens.
__device__ __forceinline__ void build_pack_index(const uint8_t* mask, int ntok, int N, int B, const IndexOut& idx) {
  constexpr int kWaves = kGateThreads / kWave;
  constexpr int kRounds = 8, kPerRound = kGateThreads * 16;
  __shared__ int s_wave[2][kWaves];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
  int carry = 0;                                       // selected tokens before the round (the same in every thread)
  const int tail = ntok & ~3;                          // start of the one partial word at the end of the mask
  for (int t_super = 0; t_super < ntok; t_super += kRounds * kPerRound) {
    uint32_t m[kRounds][4];
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        m[r][k] = 0u;
        const int tk = t_super + r * kPerRound + tid * 16 + 4 * k;
        if (tk + 4 <= ntok)
          m[r][k] = __hip_atomic_load(reinterpret_cast<const uint32_t*>(mask + tk), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    if (tail < ntok) {                                 // the partial word, by the thread that owns it
#pragma unroll
      for (int r = 0; r < kRounds; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (t_super + r * kPerRound + tid * 16 + 4 * k == tail) {
            uint32_t word = 0u;
            for (int j = 0; j < ntok - tail; ++j)
              word |= (uint32_t)__hip_atomic_load(mask + tail + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) << (8 * j);
            m[r][k] = word;
          }
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const int t0 = t_super + r * kPerRound + tid * 16;
      if (t_super + r * kPerRound >= ntok) break;      // uniform
      const int cnt = nonzero_bytes_u32(m[r][0]) + nonzero_bytes_u32(m[r][1]) + nonzero_bytes_u32(m[r][2]) +
                      nonzero_bytes_u32(m[r][3]);
      const int inc = wave_scan(cnt);
      if (lane == kWave - 1) s_wave[r & 1][wv] = inc;
      __syncthreads();                                 // one barrier per round: the wave totals alternate between two rows
      int run = carry + inc - cnt, total = 0;          // selected tokens before this thread's first token
#pragma unroll
      for (int i = 0; i < kWaves; ++i) {
        const int c = s_wave[r & 1][i];
        if (i < wv) run += c;
        total += c;
      }
      carry += total;
      if (t0 < ntok) {
        int b = t0 / N, rr = t0 - b * N;
        int inv[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const int tok = t0 + k;
          const bool sel = ((m[r][k >> 2] >> (8 * (k & 3))) & 0xFFu) != 0u;   // bytes past ntok are zero: never selected
          if (tok < ntok && rr == 0) idx.cu_seqlens[b] = run;
          inv[k] = -1;
          if (sel) {
            idx.gather_idx[run] = tok;
            inv[k] = run;
            ++run;
          }
          if (++rr == N) { rr = 0; ++b; }
        }
        if (t0 + 16 <= ntok) {
#pragma unroll
          for (int k = 0; k < 16; k += 4) {
            const uintx4 v = {(uint32_t)inv[k], (uint32_t)inv[k + 1], (uint32_t)inv[k + 2], (uint32_t)inv[k + 3]};
            *reinterpret_cast<uintx4*>(idx.inv_pos + t0 + k) = v;
          }
        } else {
          for (int k = 0; k < ntok - t0; ++k) idx.inv_pos[t0 + k] = inv[k];
        }
      }
    }
  }
  if (tid == 0) {
    idx.cu_seqlens[B] = carry;
    if (idx.total != nullptr) idx.total[0] = carry;
  }
  if (idx.counts != nullptr) {                       // counts[b] = cu[b+1] - cu[b], from this workgroup's own writes
    __syncthreads();
    for (int b = tid; b < B; b += kGateThreads) idx.counts[b] = idx.cu_seqlens[b + 1] - idx.cu_seqlens[b];
  }
}

// Held to eight waves per SIMD (left alone the sixteen-lane form takes 74 registers: 6 waves, 1 % of a detection step).
template <typename T, int G, bool kPool, bool kIndex>
__global__ void __launch_bounds__(kGateThreads) __attribute__((amdgpu_waves_per_eu(kIndex ? 4 : 8)))
gate_select_kernel(const T* __restrict__ x, const T* __restrict__ w, float bias,
                   const float* __restrict__ s_up, const float* __restrict__ noise, float theta, int ntok, int N, int C,
                   PoolGrid pool, float* __restrict__ scores, uint8_t* __restrict__ mask, IndexOut idx) {
  constexpr int VE = Vec16<T>::kElems;
  constexpr int kGroups = kGateThreads / G;
  const int grp = threadIdx.x / G;
  const int gl = threadIdx.x % G;
  const int chunks = C / VE;
  static_assert(kGroups % 4 == 0, "a pass of the workgroup covers whole 4-token words of the mask");
  __shared__ uint8_t s_sel[kGroups];
  for (long base = (long)blockIdx.x * kGroups; base < ntok; base += (long)gridDim.x * kGroups) {
    const long tok = base + grp;
    constexpr int A = gate_chains(G);
    float acc[A] = {};
    if (tok < ntok) {
      // the lane's chunks of w come from memory like its chunks of the row (w is a few KB that every
      // workgroup reads: cache hits), issued together with them: no staging of w in LDS, no barrier
      // between the launch and the first row load
      const T* row = x + tok * (long)C;
#pragma unroll(4 / A)
      for (int c0 = 0; c0 < chunks; c0 += A * G) {
        typename Raw16<T>::type xr[A], wr[A];
#pragma unroll
        for (int a = 0; a < A; ++a) {
          const int ch = c0 + a * G + gl;
          xr[a] = {};                                      // (past the row: zeros, which change no sum)
          wr[a] = {};
          if (ch < chunks) {
            xr[a] = *reinterpret_cast<const typename Raw16<T>::type*>(row + ch * VE);
            wr[a] = *reinterpret_cast<const typename Raw16<T>::type*>(w + ch * VE);
          }
        }
#pragma unroll
        for (int a = 0; a < A; ++a)
          if (c0 + a * G < chunks) {                       // uniform
            float f[VE], wv[VE];
            widen(xr[a], f);
            widen(wr[a], wv);
#pragma unroll
            for (int i = 0; i < VE; ++i) acc[a] = fmaf(f[i], wv[i], acc[a]);
          }
      }
    }
    const float dot = group_sum<G>(fold_chains(acc));
    if (gl == 0 && tok < ntok) {
      float s = dot + bias;
      if (kPool) {
        const int b = (int)(tok / N), n = (int)(tok - (long)b * N);
        const int oy = n / pool.gw, ox = n - oy * pool.gw;
        const float* p = s_up + (long)b * N * 4 + (long)(2 * oy) * (2 * pool.gw) + 2 * ox;
        const float2 top = *reinterpret_cast<const float2*>(p);
        const float2 bot = *reinterpret_cast<const float2*>(p + 2 * pool.gw);
        const float up = fmaxf(fmaxf(top.x, top.y), fmaxf(bot.x, bot.y));
        if (pool.s_up_pooled != nullptr) pool.s_up_pooled[tok] = up;
        s = fmaxf(s, up);
      } else if (s_up != nullptr) {
        s = fmaxf(s, s_up[tok]);
      }
      // noise: logistic variate of the two-class Gumbel-Softmax; theta already carries the temperature
      const bool sel = (noise != nullptr ? s + noise[tok] : s) > theta;
      scores[tok] = s;
      if (kIndex) s_sel[grp] = sel ? 1 : 0;
      else mask[tok] = sel ? 1 : 0;
    }
    if (kIndex) {
      // With the index built in this launch the mask is written with agent-scope stores, whole
      // 4-token words (byte stores past the caches cost a partial write to memory each): such a
      // store goes through the XCD's write-back L2, so that the last workgroup, on whatever XCD it
      // runs, reads the bytes without any workgroup having to flush its L2.  The pass covers tokens
      // [base, base + kGroups), base a multiple of 4; the mask is 16-byte aligned.
      __syncthreads();
      if (threadIdx.x < kGroups / 4) {
        const long t4 = base + 4 * threadIdx.x;
        if (t4 + 4 <= ntok) {
          const uint32_t word = (uint32_t)s_sel[4 * threadIdx.x] | ((uint32_t)s_sel[4 * threadIdx.x + 1] << 8) |
                                ((uint32_t)s_sel[4 * threadIdx.x + 2] << 16) | ((uint32_t)s_sel[4 * threadIdx.x + 3] << 24);
          __hip_atomic_store(reinterpret_cast<uint32_t*>(mask + t4), word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
          for (long t = t4; t < ntok; ++t)
            __hip_atomic_store(mask + t, s_sel[t - base], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_s_waitcnt(0);               // the stores have completed before this thread goes on
      }
      __syncthreads();
    }
  }
  if (kIndex) {
    // sign off: this workgroup's mask stores have completed (see above; the barrier that ends the
    // last pass orders them before what follows) before its arrival is counted; the workgroup whose
    // arrival completes the count reads the mask with agent-scope loads and builds the index.  No
    // workgroup waits for another.
    __shared__ int s_last;
    if (threadIdx.x == 0) {
      const unsigned g = blockIdx.x % kArriveGroups, groups = min((unsigned)kArriveGroups, gridDim.x);
      const unsigned members = (gridDim.x - g + kArriveGroups - 1) / kArriveGroups;      // workgroups of group g
      unsigned* mine = idx.arrive + (1 + g) * kArriveStride;
      int last = 0;
      if (atomicAdd(mine, 1u) == members - 1) {      // last of its group: nobody touches this counter again
        __hip_atomic_store(mine, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (atomicAdd(idx.arrive, 1u) == groups - 1) {
          __hip_atomic_store(idx.arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // counters left as found
          last = 1;
        }
      }
      s_last = last;
    }
    __syncthreads();
    if (s_last) build_pack_index(mask, ntok, N, ntok / N, idx);
  }
}

// ---- the gates of a hierarchy in one launch (launch groups) -----------------------------------
// Stage i's score is the larger of its own gate and the 2x2 max-pooled scores of stage i - 1 (twice as fine).  A
// workgroup takes kPyramidTokens / 4^(L-1) neighbouring tokens of the coarsest of the L stages and every token of the
// finer ones that they cover: the rows of all of them are independent loads and dot products, and the scores a
// stage hands to the next stay in LDS.  Each token's sum is the one gate_select_kernel forms, lane for lane.
// Four dependent launches of 4-5 us each for 20 MB of rows before; see spa_group_begin.
struct GateStage {
  const __bf16 *x, *w;
  float bias, theta;
  int ntok, N, C, gw;              // gw: 0 for the finest stage
  const float* s_up;
  float *scores, *s_up_pooled;
  uint8_t* mask;
};
constexpr int kPyramidTokens = 64;                       // of the finest stage, per workgroup
struct PyramidArgs {
  GateStage st[kGroupMax];
  int L;
};
// Dot products of tokens 0 .. n-1 (rows named by at(i)) with w into out[], by the groups of G lanes of `threads`
// threads, this one being number `tid`: U tokens of a group and K chunks of each in flight together.
template <int G, int U, int K, class At>
__device__ __forceinline__ void pyramid_dots(const GateStage& s, int n, float* out, int tid, int threads, At at) {
  constexpr int VE = 8, A = gate_chains(G) < K ? gate_chains(G) : K;       // (K chunks of a lane are all it has, or a multiple of the chains)
  const int grp = tid / G, gl = tid % G, groups = threads / G, chunks = s.C / VE;
  for (int i0 = grp; i0 < n; i0 += groups * U) {
    const __bf16* row[U];
    float acc[U][A] = {};
#pragma unroll
    for (int u = 0; u < U; ++u) row[u] = s.x + (long)at(min(i0 + u * groups, n - 1)) * s.C;
    for (int c0 = gl; c0 < chunks; c0 += G * K) {
      bf16x8 f[K][U], wv[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int ch = min(c0 + k * G, chunks - 1);          // (past the row: a chunk again, not added)
#pragma unroll
        for (int u = 0; u < U; ++u) f[k][u] = *reinterpret_cast<const bf16x8*>(row[u] + ch * VE);
        wv[k] = *reinterpret_cast<const bf16x8*>(s.w + ch * VE);
      }
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (k == 0 || c0 + k * G < chunks) {
          const floatx8 wf = bf16x8_to_float(wv[k]);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const floatx8 xf = bf16x8_to_float(f[k][u]);
#pragma unroll
            for (int e = 0; e < VE; ++e) acc[u][k % A] = fmaf(xf[e], wf[e], acc[u][k % A]);
          }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float d = group_sum<G>(fold_chains(acc[u]));
      if (gl == 0 && i0 + u * groups < n) out[i0 + u * groups] = d;
    }
  }
}

__global__ void __launch_bounds__(kGateThreads) gate_pyramid_kernel(const PyramidArgs p) {
  __shared__ float s_score[2 * kPyramidTokens];          // the stages one after the other: 64 + 16 + 4 + 1 tokens, or fewer
  __shared__ int s_pos[kPyramidTokens / 4][3];           // image, row and column of the coarsest tokens
  const int L = p.L, R = kPyramidTokens >> (2 * (L - 1));                    // R coarsest tokens
  const GateStage& c = p.st[L - 1];
  const unsigned c0 = blockIdx.x * R;
  const int live = min(R, c.ntok - (int)c0);             // of them inside the batch
  if ((int)threadIdx.x < live) {
    const unsigned ct = c0 + threadIdx.x, b = ct / (unsigned)c.N, n = ct - b * c.N, y = n / (unsigned)c.gw;
    s_pos[threadIdx.x][0] = b;
    s_pos[threadIdx.x][1] = y;
    s_pos[threadIdx.x][2] = n - y * c.gw;
  }
  __syncthreads();
  // flat token of stage i that is number k of the workgroup's: k = (coarsest token, row, column inside its square)
  auto token = [&](int i, int k) {
    const int sh = L - 1 - i;
    const int* pos = s_pos[k >> (2 * sh)];
    const int in = k & ((1 << (2 * sh)) - 1), y = (pos[1] << sh) + (in >> sh), x = (pos[2] << sh) + (in & ((1 << sh) - 1));
    return pos[0] * p.st[i].N + y * (c.gw << sh) + x;
  };
  // the finest stage to two waves, the next to one (two stages: two), the rest to the last
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int from = 0;
  // The fourth wave has two stages, i.e. two trips to memory one after the other (2 us of 8): the line of every 64 columns of its second
  // one's token is on its way during the first.  16 images of 56 x 56 .. 7 x 7 tokens, 18 MB: 8.4 -> 8.0 us with that and the end below.
  uint32_t early = 0;
  if (L == 4 && wave == 3 && live > 0) {
    const GateStage& s = p.st[3];
    const int at = (threadIdx.x & (kWave - 1)) * 64;
    if (at < s.C) early = *reinterpret_cast<const uint32_t*>(s.x + (long)token(3, 0) * s.C + at);
  }
  for (int i = 0; i < L; ++i) {
    const GateStage& s = p.st[i];
    const int n = live << (2 * (L - 1 - i));
    const int w0 = i == 0 ? 0 : i == 1 ? 2 : 3, nw = i == 0 || L == 2 ? 2 : 1;
    if (wave >= w0 && wave < w0 + nw) {
      const int tid = threadIdx.x - w0 * kWave, nt = nw * kWave, chunks = s.C / 8;
      float* out = s_score + from;
      auto row = [&](int k) { return token(i, k); };
      switch (gate_lanes(chunks)) {
        case 8: pyramid_dots<8, 8, 1>(s, n, out, tid, nt, row); break;
        case 16:
          if (chunks <= 16) pyramid_dots<16, 8, 1>(s, n, out, tid, nt, row);
          else if (chunks <= 32) pyramid_dots<16, 4, 2>(s, n, out, tid, nt, row);
          else pyramid_dots<16, 2, 4>(s, n, out, tid, nt, row);
          break;
        case 32: pyramid_dots<32, 2, 4>(s, n, out, tid, nt, row); break;
        default: pyramid_dots<64, 2, 4>(s, n, out, tid, nt, row); break;
      }
    }
    from += n;
  }
  asm volatile("" ::"v"(early));
  __syncthreads();
  if (wave != 0) return;             // (no stage has more than 64 tokens here: one wave, whose LDS operations are in order)
  static_assert(kPyramidTokens <= kWave, "a token a lane");
  const float* finer = s_score;
  float* mine = s_score;
  for (int i = 0; i < L; ++i) {
    const GateStage& s = p.st[i];
    const int sh = L - 1 - i, n = live << (2 * sh);
    if ((int)threadIdx.x < n) {
      const int k = threadIdx.x;
      float v = mine[k] + s.bias;
      const int tok = token(i, k);
      if (i > 0) {
        // children: a square twice as wide, same coarsest token
        const int in = k & ((1 << (2 * sh)) - 1), y = in >> sh, x = in & ((1 << sh) - 1), wide = 2 << sh;
        const float* f = finer + ((k >> (2 * sh)) << (2 * sh + 2)) + 2 * y * wide + 2 * x;
        const float up = fmaxf(fmaxf(f[0], f[1]), fmaxf(f[wide], f[wide + 1]));
        if (s.s_up_pooled != nullptr) s.s_up_pooled[tok] = up;
        v = fmaxf(v, up);
      }
      s.scores[tok] = v;
      s.mask[tok] = v > s.theta ? 1 : 0;
      mine[k] = v;
    }
    finer = mine;
    mine += n;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // (other lanes read mine: an order for the compiler, no instruction)
    __builtin_amdgcn_wave_barrier();
  }
}

static thread_local Noted<GateStage> g_noted;

// counts[b] = selected tokens of image b: one workgroup per image, no atomics.
__global__ void __launch_bounds__(256)
count_selected_kernel(const uint8_t* __restrict__ mask, int N, int32_t* __restrict__ counts) {
  __shared__ int red[4];
  const uint8_t* m = mask + (long)blockIdx.x * N;
  int c = 0;
  for (int i = threadIdx.x; i < N; i += 256) c += m[i] != 0;
  c = wave_sum(c);
  if (lane_id() == 0) red[threadIdx.x / kWave] = c;
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ void maxpool2x2_kernel(const float* __restrict__ s, int B, int h, int w,
                                  float* __restrict__ out) {
  const int ho = h / 2, wo = w / 2;
  const long n = (long)B * ho * wo;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    const int b = i / (ho * wo);
    const int r = i % (ho * wo);
    const int oy = r / wo, ox = r % wo;
    const float* p = s + (long)b * h * w + (long)(2 * oy) * w + 2 * ox;
    out[i] = fmaxf(fmaxf(p[0], p[1]), fmaxf(p[w], p[w + 1]));
  }
}


// ---------------------------------------------------------------------- gate backward
// Selection loss (binary cross-entropy on sigmoid(s)) + gradient of r_g = sigmoid(s) . r.
// G lanes own a token (IT chunks of its row each), so x and d_rg are read once; every workgroup has a
// contiguous share of the tokens and a group takes U of them at a time, all their loads in flight
// together.  A row is spread over as many lanes as it has chunks (up to a wave): the dw accumulators
// are then IT * 8 registers and the fold of a workgroup is one row per wave.  With 16 lanes per token at
// every width it was 16 rows of C, 49 KB of LDS at C 768, and took as long as the token loop: 12544
// tokens of 768: 17.9 -> 15.4 us (58 MB); 50176 of 96: 13.2 -> 10.2; 784 of 768: 10.4 -> 8.0.
// dw / db / loss are reduced without atomics, in a fixed order: lanes over their tokens, the groups of a
// wave by exchanges, waves through LDS, every workgroup writes one partial row, and a second kernel adds
// the partial rows.
// Straight-through estimator of the hard selection: selected tokens differentiate the relaxed
// weight sigmoid((s + noise) / T) in place of the 0/1 mask.  mask == nullptr: off.
struct StraightThrough {
  const uint8_t* mask;
  const float* noise;   // may be null (noise-free selection)
  float inv_temperature;
};

template <typename T>
struct GateBwdArgs {
  const T *x, *w;
  float bias;
  const float *scores, *s_up;
  const uint8_t* labels;
  const T* d_rg;
  int gate_scaled;
  float loss_scale;
  StraightThrough st;
  int ntok, C;
  T* dx;
  float* partial;
};
template <typename T, int G, int IT, int U>
__device__ __forceinline__ void gate_bwd_block(const GateBwdArgs<T>& a, unsigned block, unsigned blocks, float* lds) {
  constexpr int VE = Vec16<T>::kElems, kGroups = kGateThreads / G, kWaves = kGateThreads / kWave;
  using Raw = typename Raw16<T>::type;
  __shared__ float s_loss[kWaves], s_db[kWaves];
  const T *x = a.x, *w = a.w, *d_rg = a.d_rg;
  const float *scores = a.scores, *s_up = a.s_up;
  const uint8_t* labels = a.labels;
  const float bias = a.bias, loss_scale = a.loss_scale;
  const StraightThrough st = a.st;
  const int ntok = a.ntok, C = a.C, gate_scaled = a.gate_scaled;
  T* dx = a.dx;
  float* partial = a.partial;

  const int grp = threadIdx.x / G, gl = threadIdx.x % G;
  const int chunks = C / VE;
  const bool scaled = gate_scaled != 0 && d_rg != nullptr;
  float wv[IT][VE], dwa[IT][VE];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int ch = gl + it * G;
    Raw r = {};
    if (ch < chunks) r = *reinterpret_cast<const Raw*>(w + ch * VE);
    widen(r, wv[it]);
#pragma unroll
    for (int e = 0; e < VE; ++e) dwa[it][e] = 0.f;
  }
  float loss_acc = 0.f, db_acc = 0.f;

  const long per = ((long)ntok + blocks - 1) / blocks;
  const long t0 = block * per, t1 = min((long)ntok, t0 + per);
  for (long base = t0 + grp; base < t1; base += kGroups * U) {
    Raw xr[U][IT], dr[U][IT];
    float s[U], up[U], nz[U];
    uint8_t lab[U], sel[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long tok = min(base + u * kGroups, t1 - 1);      // past the share: a valid token, its results unused
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int ch = gl + it * G;
        xr[u][it] = {};
        dr[u][it] = {};
        if (ch < chunks) {
          xr[u][it] = *reinterpret_cast<const Raw*>(x + tok * C + ch * VE);
          if (scaled) dr[u][it] = *reinterpret_cast<const Raw*>(d_rg + tok * C + ch * VE);
        }
      }
      s[u] = scores[tok];
      lab[u] = labels[tok];
      up[u] = s_up != nullptr ? s_up[tok] : 0.f;
      sel[u] = st.mask != nullptr ? st.mask[tok] : 0;
      nz[u] = st.noise != nullptr ? st.noise[tok] : 0.f;
    }
    float s_mine = 0.f, y_mine = 0.f, d_mine = 0.f;          // lane u of the group keeps the loss of its token u
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long tok = base + u * kGroups;
      float xf[IT][VE], df[IT][VE];
      float dot = 0.f;
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        widen(xr[u][it], xf[it]);
        widen(dr[u][it], df[it]);
#pragma unroll
        for (int e = 0; e < VE; ++e) dot = fmaf(df[it][e], xf[it][e], dot);
      }
      dot = group_sum<G>(dot);
      bool own = tok < t1;
      if (s_up != nullptr) {                             // (uniform) did the up-scale score win the max? (see gate_chains)
        float g = 0.f;
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
          for (int e = 0; e < VE; ++e) g = fmaf(xf[it][e], wv[it][e], g);
        own = own && group_sum<G>(g) + bias >= up[u];
      }
      const float p = sigmoidf_dev(s[u]);
      const float y = lab[u] != 0 ? 1.f : 0.f;
      float ds = loss_scale * (p - y);
      if (scaled) {
        float coef = p * (1.f - p);                      // through r_g = sigmoid(s) . r
        if (sel[u] != 0) {                               // through the relaxed selection weight: <d_rg, r_g> = p dot
          const float pt = sigmoidf_dev((s[u] + nz[u]) * st.inv_temperature);
          coef = fmaf(pt * (1.f - pt) * st.inv_temperature, p, coef);
        }
        ds = fmaf(coef, dot, ds);
      }
      const float dsg = own ? ds : 0.f;                  // (w, b) get no gradient where the up-scale score won
      const float pg = scaled ? p : 0.f;
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int ch = gl + it * G;
        float o[VE];
#pragma unroll
        for (int e = 0; e < VE; ++e) {
          o[e] = fmaf(dsg, wv[it][e], pg * df[it][e]);
          dwa[it][e] = fmaf(dsg, xf[it][e], dwa[it][e]);
        }
        if (ch < chunks && tok < t1) Vec16<T>::store(dx + tok * C + ch * VE, o);
      }
      if (gl == u) { s_mine = s[u]; y_mine = y; d_mine = dsg; }
    }
    if (gl < U && base + gl * kGroups < t1) {
      loss_acc += fmaxf(s_mine, 0.f) - y_mine * s_mine + log1pf(__expf(-fabsf(s_mine)));
      db_acc += d_mine;
    }
  }

  // fold: the groups of a wave by exchanges, then one row per wave
#pragma unroll
  for (int it = 0; it < IT; ++it)
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      if (G <= 16) dwa[it][e] = add_lane_xor16(dwa[it][e]);
      if (G <= 32) dwa[it][e] = add_lane_xor32(dwa[it][e]);
    }
  loss_acc = group_sum<kWave>(loss_acc);
  db_acc = group_sum<kWave>(db_acc);
  const int wv_id = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) < G) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int ch = gl + it * G;
      if (ch < chunks) {
#pragma unroll
        for (int e = 0; e < VE; e += 4) {
          const floatx4 f = {dwa[it][e], dwa[it][e + 1], dwa[it][e + 2], dwa[it][e + 3]};
          *reinterpret_cast<floatx4*>(&lds[wv_id * C + ch * VE + e]) = f;
        }
      }
    }
  }
  if ((threadIdx.x & (kWave - 1)) == 0) { s_loss[wv_id] = loss_acc; s_db[wv_id] = db_acc; }
  __syncthreads();
  float* prow = partial + (long)block * (C + 2);
  for (int c = threadIdx.x; c < C; c += kGateThreads) {
    float a = 0.f;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) a += lds[i * C + c];
    prow[c] = a;
  }
  if (threadIdx.x == 0) {
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) { a += s_loss[i]; b += s_db[i]; }
    prow[C] = a;
    prow[C + 1] = b;
  }
}

// LDS: 4 rows of C floats
template <typename T, int G, int IT, int U>
__global__ void __launch_bounds__(kGateThreads) gate_bwd_kernel(const GateBwdArgs<T> a) {
  extern __shared__ float lds[];
  gate_bwd_block<T, G, IT, U>(a, blockIdx.x, gridDim.x, lds);
}
// Several calls in one launch (launch groups): the forms of launch_gate_bwd, up to 1024 columns
__global__ void __launch_bounds__(kGateThreads) gate_bwd_group_kernel(const Members<GateBwdArgs<__bf16>> m) {
  extern __shared__ float lds[];
  const MemberBlock mb = member_of(m, blockIdx.x);
  const GateBwdArgs<__bf16>& a = m.a[mb.s];
  const int chunks = a.C / 8;
  if (chunks <= 16) gate_bwd_block<__bf16, 16, 1, 4>(a, mb.block, mb.blocks, lds);
  else if (chunks <= 32) gate_bwd_block<__bf16, 32, 1, 4>(a, mb.block, mb.blocks, lds);
  else if (chunks <= 64) gate_bwd_block<__bf16, 64, 1, 4>(a, mb.block, mb.blocks, lds);
  else gate_bwd_block<__bf16, 64, 2, 4>(a, mb.block, mb.blocks, lds);
}

// Adds the partial rows in a fixed order: a block owns 16 columns; SL row slices run in parallel
// (slice s adds rows s, s+SL, ..., at most 8 of them, whose loads are all in flight at once), then the
// slices of a wave are added by exchanges and the waves in order.  64 slices, or 16 where these reach all rows
// (at most 128): sixteen waves a workgroup start later than four, 0.6 us of the 7.6 of both launches at 50 tokens of 64.
constexpr int kGateBwdMaxParts = 512;
struct GateReduceArgs {
  const float* partial;
  int nparts, C;
  float loss_scale;
  float *loss, *dw, *db;
};
template <int SL>
__device__ __forceinline__ void gate_bwd_reduce_block(const GateReduceArgs& g, int block) {
  constexpr int kRows = 8, kWaves = SL / 4;
  static_assert(kGateBwdMaxParts <= 64 * kRows, "64 slices reach every row");
  const float* partial = g.partial;
  const int nparts = g.nparts, C = g.C;
  __shared__ float red[kWaves][17];
  const int cl = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int c = block * 16 + cl;
  float v[kRows];
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const int r = sl + SL * i;
    v[i] = r < nparts && c < C + 2 ? partial[(long)r * (C + 2) + c] : 0.f;
  }
  float a = 0.f;
#pragma unroll
  for (int i = 0; i < kRows; ++i) a += v[i];
  a = add_lane_xor32(add_lane_xor16(a));
  if ((threadIdx.x & 63) < 16) red[threadIdx.x >> 6][cl] = a;
  __syncthreads();
  if (threadIdx.x < 16 && c < C + 2) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) t += red[i][cl];
    if (c < C) g.dw[c] = t;
    else if (c == C) g.loss[0] = t * g.loss_scale;
    else g.db[0] = t;
  }
}
template <int SL>
__global__ void __launch_bounds__(16 * SL) gate_bwd_reduce_kernel(const GateReduceArgs g) {
  gate_bwd_reduce_block<SL>(g, blockIdx.x);
}
__global__ void __launch_bounds__(1024) gate_bwd_reduce_group_kernel(const Members<GateReduceArgs> m) {
  const MemberBlock mb = member_of(m, blockIdx.x);
  gate_bwd_reduce_block<64>(m.a[mb.s], mb.block);
}

static thread_local Noted<GateBwdArgs<__bf16>> g_noted_bwd;
static thread_local Noted<GateReduceArgs> g_noted_reduce;
void group_forget_gates() { g_noted.n = g_noted_bwd.n = g_noted_reduce.n = 0; }
int group_flush_gates_bwd(hipStream_t st) {
  if (g_noted_bwd.n == 0) return SPA_OK;
  int C = 0;
  for (int i = 0; i < g_noted_bwd.n; ++i) C = std::max(C, g_noted_bwd.a[i].C);
  Members<GateBwdArgs<__bf16>> m;
  const unsigned blocks = g_noted_bwd.members(m);
  hipLaunchKernelGGL(gate_bwd_group_kernel, dim3(blocks), dim3(kGateThreads), (kGateThreads / kWave) * C * sizeof(float), st, m);
  Members<GateReduceArgs> r;
  const unsigned rblocks = g_noted_reduce.members(r);
  hipLaunchKernelGGL(gate_bwd_reduce_group_kernel, dim3(rblocks), dim3(1024), 0, st, r);
  return check_launch("spa_group_end");
}

static int gate_bwd_parts(long ntok) {
  long p = (ntok + 15) / 16;
  if (p > kGateBwdMaxParts) p = kGateBwdMaxParts;
  if (p < 1) p = 1;
  return (int)p;
}

template <typename T>
static int launch_gate(const char* fn, const void* x, const void* w, float bias, const float* s_up,
                       const float* noise, float theta, int B, int N, int C, PoolGrid pool, bool pooled,
                       float* scores, uint8_t* mask, int32_t* counts, hipStream_t st,
                       IndexOut idx = IndexOut{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr}) {
  constexpr int VE = Vec16<T>::kElems;
  const int chunks = C / VE;
  const long ntok = (long)B * N;
  const size_t lds = 0;      // (the gate weight is read from memory, nothing is staged)
  auto go = [&](auto gtag) {
    constexpr int G = decltype(gtag)::value;
    const long per_wg = kGateThreads / G;
    long wgs = (ntok + per_wg - 1) / per_wg;
    if (wgs > 4096) wgs = 4096;
    if (pooled)
      hipLaunchKernelGGL((gate_select_kernel<T, G, true, false>), dim3((unsigned)wgs), dim3(kGateThreads), lds, st,
                         static_cast<const T*>(x), static_cast<const T*>(w), bias, s_up, noise, theta,
                         (int)ntok, N, C, pool, scores, mask, idx);
    else if (idx.arrive != nullptr)
      hipLaunchKernelGGL((gate_select_kernel<T, G, false, true>), dim3((unsigned)wgs), dim3(kGateThreads), lds, st,
                         static_cast<const T*>(x), static_cast<const T*>(w), bias, s_up, noise, theta,
                         (int)ntok, N, C, pool, scores, mask, idx);
    else
      hipLaunchKernelGGL((gate_select_kernel<T, G, false, false>), dim3((unsigned)wgs), dim3(kGateThreads), lds, st,
                         static_cast<const T*>(x), static_cast<const T*>(w), bias, s_up, noise, theta,
                         (int)ntok, N, C, pool, scores, mask, idx);
  };
  switch (gate_lanes(chunks)) {
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 16: go(std::integral_constant<int, 16>{}); break;
    case 32: go(std::integral_constant<int, 32>{}); break;
    default: go(std::integral_constant<int, 64>{}); break;
  }
  if (counts != nullptr && idx.arrive == nullptr)
    hipLaunchKernelGGL(count_selected_kernel, dim3(B), dim3(256), 0, st, mask, N, counts);
  return check_launch(fn);
}

// The noted gates: one launch where each takes the scores of the one before it, else one by one, in order.
int group_flush_gates(hipStream_t st) {
  const Noted<GateStage>& g = g_noted;
  bool chain = g.n >= 2 && g.a[0].gw == 0 && g.a[0].s_up == nullptr;
  for (int i = 1; i < g.n; ++i)
    chain = chain && g.a[i].gw > 0 && g.a[i].s_up == g.a[i - 1].scores && g.a[i - 1].N == 4 * g.a[i].N && g.a[i - 1].ntok == 4 * g.a[i].ntok &&
            (i == 1 || g.a[i - 1].gw == 2 * g.a[i].gw);
  if (chain) {
    PyramidArgs p;
    for (int i = 0; i < kGroupMax; ++i) p.st[i] = g.a[i < g.n ? i : g.n - 1];
    p.L = g.n;
    const long R = kPyramidTokens >> (2 * (g.n - 1)), wgs = (p.st[g.n - 1].ntok + R - 1) / R;
    hipLaunchKernelGGL(gate_pyramid_kernel, dim3((unsigned)wgs), dim3(kGateThreads), 0, st, p);
    return check_launch("spa_group_end");
  }
  for (int i = 0; i < g.n; ++i) {
    const GateStage& s = g.a[i];
    const bool pooled = s.gw > 0;
    if (int rc = launch_gate<__bf16>("spa_group_end", s.x, s.w, s.bias, s.s_up, nullptr, s.theta, s.ntok / s.N, s.N, s.C,
                                     PoolGrid{pooled ? s.N / s.gw : 0, s.gw, s.s_up_pooled}, pooled, s.scores, s.mask,
                                     nullptr, st))
      return rc;
  }
  return SPA_OK;
}

}  // namespace spa

using namespace spa;

static int gate_select_common(const char* fn, const void* x, const void* w, float bias, const float* s_up,
                              const float* noise, float temperature, float tau, int B, int N, int C, int dtype,
                              float* scores, uint8_t* mask, int32_t* counts, void* stream,
                              PoolGrid pool = PoolGrid{0, 0, nullptr}, bool pooled = false,
                              IndexOut idx = IndexOut{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr}) {
  SPA_REQUIRE(x && w && scores && mask, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(B >= 1 && N >= 1 && C >= 1, SPA_ERR_INVALID_ARG, "%s: B, N, C must be >= 1", fn);
  SPA_REQUIRE((long)B * N < 2147483647L, SPA_ERR_INVALID_ARG, "%s: B*N must be < 2^31", fn);
  SPA_REQUIRE(tau > 0.f && tau < 1.f, SPA_ERR_INVALID_ARG, "%s: tau must lie in (0,1), got %g", fn, (double)tau);
  SPA_REQUIRE(temperature > 0.f && std::isfinite(temperature), SPA_ERR_INVALID_ARG,
              "%s: temperature must be positive and finite, got %g", fn, (double)temperature);
  SPA_REQUIRE(dtype == SPA_F32 || dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: unknown dtype %d", fn, dtype);
  SPA_REQUIRE(((long)C * elem_size(dtype)) % 16 == 0, SPA_ERR_INVALID_ARG,
              "%s: row length C*elem = %ld bytes is not a multiple of 16", fn, (long)C * elem_size(dtype));
  SPA_REQUIRE(aligned16(x), SPA_ERR_INVALID_ARG, "%s: x is not 16-byte aligned", fn);
  SPA_REQUIRE(C <= kMaxGateC, SPA_ERR_UNSUPPORTED, "%s: C = %d exceeds %d", fn, C, kMaxGateC);
  // sigmoid((s + e) / T) > tau  <=>  s + e > T * logit(tau)
  const float theta = (float)((double)temperature * std::log((double)tau / (1.0 - (double)tau)));
  hipStream_t st = as_stream(stream);
  if (group_open()) {
    SPA_REQUIRE(dtype == SPA_BF16 && noise == nullptr && counts == nullptr && idx.arrive == nullptr, SPA_ERR_UNSUPPORTED,
                "%s: this form cannot be part of a group", fn);
    return g_noted.add(fn, GateStage{static_cast<const __bf16*>(x), static_cast<const __bf16*>(w), bias, theta, B * N, N, C,
                                     pooled ? pool.gw : 0, s_up, scores, pool.s_up_pooled, mask}, 0);
  }
  if (dtype == SPA_F32)
    return launch_gate<float>(fn, x, w, bias, s_up, noise, theta, B, N, C, pool, pooled, scores, mask, counts, st, idx);
  return launch_gate<__bf16>(fn, x, w, bias, s_up, noise, theta, B, N, C, pool, pooled, scores, mask, counts, st, idx);
}

extern "C" int spa_gate_select(const void* x, const void* w, float bias, const float* s_up,
                               float tau, int B, int N, int C, int dtype, float* scores,
                               uint8_t* mask, int32_t* counts, void* stream) {
  return gate_select_common("spa_gate_select", x, w, bias, s_up, nullptr, 1.f, tau, B, N, C, dtype, scores, mask,
                            counts, stream);
}

extern "C" int spa_gate_select_index(const void* x, const void* w, float bias, const float* s_up, float tau, int B,
                                     int N, int C, int dtype, float* scores, uint8_t* mask, int32_t* counts,
                                     int32_t* cu_seqlens, int32_t* gather_idx, int32_t* inv_pos, int32_t* total,
                                     void* workspace, size_t workspace_bytes, void* stream) {
  const char* fn = "spa_gate_select_index";
  SPA_REQUIRE(cu_seqlens && gather_idx && inv_pos, SPA_ERR_INVALID_ARG, "%s: null index pointer", fn);
  SPA_REQUIRE(workspace != nullptr && workspace_bytes >= kArriveWords * sizeof(unsigned), SPA_ERR_WORKSPACE,
              "%s: workspace of %zu bytes needed (zero-filled once, left zero by every call), %zu given", fn,
              kArriveWords * sizeof(unsigned), workspace_bytes);
  SPA_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 3u) == 0 && aligned16(mask) && aligned16(inv_pos),
              SPA_ERR_INVALID_ARG, "%s: mask / inv_pos not 16-byte aligned or workspace not 4-byte aligned", fn);
  const IndexOut idx = {cu_seqlens, gather_idx, inv_pos, total, counts, static_cast<unsigned*>(workspace)};
  return gate_select_common(fn, x, w, bias, s_up, nullptr, 1.f, tau, B, N, C, dtype, scores, mask, counts, stream,
                            PoolGrid{0, 0, nullptr}, false, idx);
}

extern "C" int spa_gate_select_gumbel(const void* x, const void* w, float bias, const float* s_up,
                                      const float* noise, float temperature, float tau, int B, int N, int C,
                                      int dtype, float* scores, uint8_t* mask, int32_t* counts, void* stream) {
  SPA_REQUIRE(noise != nullptr, SPA_ERR_INVALID_ARG, "spa_gate_select_gumbel: noise is null");
  return gate_select_common("spa_gate_select_gumbel", x, w, bias, s_up, noise, temperature, tau, B, N, C, dtype,
                            scores, mask, counts, stream);
}

extern "C" int spa_gate_select_pooled(const void* x, const void* w, float bias, const float* s_fine,
                                      float tau, int B, int grid_h, int grid_w, int C, int dtype, float* scores,
                                      uint8_t* mask, int32_t* counts, float* s_up_pooled, void* stream) {
  const char* fn = "spa_gate_select_pooled";
  SPA_REQUIRE(s_fine != nullptr, SPA_ERR_INVALID_ARG, "%s: s_fine is null", fn);
  SPA_REQUIRE(grid_h >= 1 && grid_w >= 1 && (long)grid_h * grid_w < 2147483647L / 4, SPA_ERR_INVALID_ARG,
              "%s: grid_h, grid_w must be >= 1", fn);
  SPA_REQUIRE((reinterpret_cast<uintptr_t>(s_fine) & 7) == 0, SPA_ERR_INVALID_ARG, "%s: s_fine not 8-byte aligned", fn);
  return gate_select_common(fn, x, w, bias, s_fine, nullptr, 1.f, tau, B, grid_h * grid_w, C, dtype, scores, mask,
                            counts, stream, PoolGrid{grid_h, grid_w, s_up_pooled}, true);
}

extern "C" int spa_maxpool2x2(const float* s, int B, int h, int w, float* pooled, void* stream) {
  SPA_REFUSE_IN_GROUP("spa_maxpool2x2");
  SPA_REQUIRE(s && pooled, SPA_ERR_INVALID_ARG, "spa_maxpool2x2: null pointer");
  SPA_REQUIRE(B >= 1 && h >= 2 && w >= 2 && h % 2 == 0 && w % 2 == 0, SPA_ERR_INVALID_ARG,
              "spa_maxpool2x2: need B >= 1 and even h, w >= 2 (got %d, %d, %d)", B, h, w);
  const long n = (long)B * (h / 2) * (w / 2);
  long wgs = (n + 255) / 256;
  if (wgs > 2048) wgs = 2048;
  hipLaunchKernelGGL(maxpool2x2_kernel, dim3((unsigned)wgs), dim3(256), 0, as_stream(stream), s, B, h, w, pooled);
  return check_launch("spa_maxpool2x2");
}

extern "C" size_t spa_gate_bwd_workspace_bytes(int B, int N, int C, int dtype) {
  (void)dtype;
  if (B < 1 || N < 1 || C < 1) return 0;
  return (size_t)gate_bwd_parts((long)B * N) * (size_t)(C + 2) * sizeof(float);
}

template <typename T>
static int launch_gate_bwd(const void* x, const void* w, float bias, const float* scores, const float* s_up,
                           const uint8_t* labels, const void* d_rg, int gate_scaled, float loss_scale,
                           StraightThrough stt, long ntok, int C, float* loss, void* dx, float* dw, float* db,
                           float* partial, hipStream_t st) {
  constexpr int VE = Vec16<T>::kElems;
  const int chunks = C / VE;
  const int parts = gate_bwd_parts(ntok);
  const size_t lds = (size_t)(kGateThreads / kWave) * C * sizeof(float);      // at most 64 KB (C <= 4096)
  const GateBwdArgs<T> args = {static_cast<const T*>(x), static_cast<const T*>(w), bias, scores, s_up, labels,
                               static_cast<const T*>(d_rg), gate_scaled, loss_scale, stt, (int)ntok, C, static_cast<T*>(dx),
                               partial};
  const GateReduceArgs rargs = {partial, parts, C, loss_scale, loss, dw, db};
  const unsigned rblocks = (C + 2 + 15) / 16;
  if constexpr (sizeof(T) == 2) {
    if (group_open()) {
      SPA_REQUIRE(C <= 1024, SPA_ERR_UNSUPPORTED, "spa_gate_bwd: C = %d > 1024 cannot be part of a group", C);
      if (int rc = g_noted_bwd.add("spa_gate_bwd", args, parts)) return rc;
      return g_noted_reduce.add("spa_gate_bwd", rargs, rblocks);
    }
  }
  SPA_REQUIRE(!group_open(), SPA_ERR_UNSUPPORTED, "spa_gate_bwd: fp32 calls cannot be part of a group");
#define SPA_GB(G, IT, U) hipLaunchKernelGGL((gate_bwd_kernel<T, G, IT, U>), dim3(parts), dim3(kGateThreads), lds, st, args)
  // (up to 512 shares a share is 16 tokens, one per group of 16 lanes, two per group of 32: no more taken at a time)
  const bool few = ntok <= 16L * kGateBwdMaxParts;
  if (chunks <= 16 && few) SPA_GB(16, 1, 1);
  else if (chunks <= 16) SPA_GB(16, 1, 4);
  else if (chunks <= 32 && few) SPA_GB(32, 1, 2);
  else if (chunks <= 32) SPA_GB(32, 1, 4);
  else if (chunks <= 64) SPA_GB(64, 1, 4);
  else if (chunks <= 128) SPA_GB(64, 2, 4);
  else if (chunks <= 256) SPA_GB(64, 4, 2);
  else if (chunks <= 512) SPA_GB(64, 8, 1);
  else return fail(SPA_ERR_UNSUPPORTED, "spa_gate_bwd: C = %d too large (at most %d)", C, 512 * VE);
#undef SPA_GB
  if (parts <= 128) hipLaunchKernelGGL(gate_bwd_reduce_kernel<16>, dim3(rblocks), dim3(256), 0, st, rargs);
  else hipLaunchKernelGGL(gate_bwd_reduce_kernel<64>, dim3(rblocks), dim3(1024), 0, st, rargs);
  return check_launch("spa_gate_bwd");
}

static int gate_bwd_common(const char* fn, const void* x, const void* w, float bias, const float* scores,
                           const float* s_up, const uint8_t* labels, const void* d_rg, int gate_scaled,
                           float loss_scale, StraightThrough stt, int B, int N, int C, int dtype, float* loss,
                           void* dx, float* dw, float* db, void* workspace, size_t workspace_bytes, void* stream) {
  SPA_REQUIRE(x && w && scores && labels && loss && dx && dw && db, SPA_ERR_INVALID_ARG, "%s: null pointer", fn);
  SPA_REQUIRE(B >= 1 && N >= 1 && C >= 1, SPA_ERR_INVALID_ARG, "%s: B, N, C must be >= 1", fn);
  SPA_REQUIRE((long)B * N < 2147483647L, SPA_ERR_INVALID_ARG, "%s: B*N must be < 2^31", fn);
  SPA_REQUIRE(dtype == SPA_F32 || dtype == SPA_BF16, SPA_ERR_UNSUPPORTED, "%s: unknown dtype %d", fn, dtype);
  SPA_REQUIRE(((long)C * elem_size(dtype)) % 16 == 0, SPA_ERR_INVALID_ARG,
              "%s: row length C*elem = %ld bytes is not a multiple of 16", fn, (long)C * elem_size(dtype));
  SPA_REQUIRE(aligned16(x) && aligned16(dx) && aligned16(d_rg), SPA_ERR_INVALID_ARG,
              "%s: x / dx / d_rg not 16-byte aligned", fn);
  SPA_REQUIRE(!(gate_scaled && !d_rg), SPA_ERR_INVALID_ARG, "%s: gate_scaled needs d_rg", fn);
  SPA_REQUIRE(C <= kMaxGateC, SPA_ERR_UNSUPPORTED, "%s: C = %d exceeds %d", fn, C, kMaxGateC);
  const size_t need = spa_gate_bwd_workspace_bytes(B, N, C, dtype);
  SPA_REQUIRE(workspace != nullptr && workspace_bytes >= need, SPA_ERR_WORKSPACE,
              "%s: workspace of %zu bytes needed, %zu given", fn, need, workspace_bytes);
  hipStream_t st = as_stream(stream);
  float* partial = static_cast<float*>(workspace);
  if (dtype == SPA_F32)
    return launch_gate_bwd<float>(x, w, bias, scores, s_up, labels, d_rg, gate_scaled, loss_scale, stt, (long)B * N,
                                  C, loss, dx, dw, db, partial, st);
  return launch_gate_bwd<__bf16>(x, w, bias, scores, s_up, labels, d_rg, gate_scaled, loss_scale, stt, (long)B * N,
                                 C, loss, dx, dw, db, partial, st);
}

extern "C" int spa_gate_bwd(const void* x, const void* w, float bias, const float* scores,
                            const float* s_up, const uint8_t* labels, const void* d_rg, int gate_scaled,
                            float loss_scale, int B, int N, int C, int dtype, float* loss, void* dx,
                            float* dw, float* db, void* workspace, size_t workspace_bytes, void* stream) {
  return gate_bwd_common("spa_gate_bwd", x, w, bias, scores, s_up, labels, d_rg, gate_scaled, loss_scale,
                         StraightThrough{nullptr, nullptr, 1.f}, B, N, C, dtype, loss, dx, dw, db, workspace,
                         workspace_bytes, stream);
}

// ---- the gate backward for callers that cannot allocate --------------------------------
// The partial rows of the two-stage reduction live in a file-scope device array instead of a
// caller workspace.  The array's name is a host-side stand-in, not a device address: its
// address on the current device is looked up once per device with hipGetSymbolAddress and that
// pointer is what the kernels get.
namespace spa {
constexpr int kNoAllocMaxC = 1024;
constexpr int kNoAllocMaxDevices = 64;
static __device__ __align__(256) float scratch[(size_t)kGateBwdMaxParts * (kNoAllocMaxC + 2)];
static float* g_scratch_ptr[kNoAllocMaxDevices] = {};
static std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device (looked up on the first call on that device).
static int scratch_on_current_device(const char* fn, float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(SPA_ERR_HIP, "%s: hipGetDevice: %s", fn, hipGetErrorString(e));
  SPA_REQUIRE(dev >= 0 && dev < kNoAllocMaxDevices, SPA_ERR_UNSUPPORTED, "%s: device %d beyond %d", fn, dev,
              kNoAllocMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      return fail(SPA_ERR_HIP, "%s: hipGetSymbolAddress(scratch): %s", fn, hipGetErrorString(e));
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return SPA_OK;
}
}  // namespace spa

extern "C" int spa_gate_bwd_static(const void* x, const void* w, float bias, const float* scores,
                                   const float* s_up, const uint8_t* labels, const void* d_rg, int gate_scaled,
                                   float loss_scale, int B, int N, int C, int dtype, float* loss, void* dx,
                                   float* dw, float* db, void* stream) {
  const char* fn = "spa_gate_bwd_static";
  SPA_REQUIRE(C >= 1 && C <= kNoAllocMaxC, SPA_ERR_WORKSPACE,
              "%s: C = %d exceeds the built-in scratch (C <= %d); use spa_gate_bwd with a workspace", fn, C,
              kNoAllocMaxC);
  SPA_REQUIRE(B >= 1 && N >= 1, SPA_ERR_INVALID_ARG, "%s: B, N must be >= 1", fn);
  const size_t need = spa_gate_bwd_workspace_bytes(B, N, C, dtype);
  SPA_REQUIRE(need <= sizeof(float) * (size_t)kGateBwdMaxParts * (kNoAllocMaxC + 2), SPA_ERR_WORKSPACE,
              "%s: %zu bytes of scratch needed, more than the built-in array holds", fn, need);
  float* ptr = nullptr;
  if (int rc = scratch_on_current_device(fn, &ptr)) return rc;
  // every partial row the reduction reads is written by this call's first kernel: nothing to clear
  return gate_bwd_common(fn, x, w, bias, scores, s_up, labels, d_rg, gate_scaled, loss_scale,
                         StraightThrough{nullptr, nullptr, 1.f}, B, N, C, dtype, loss, dx, dw, db, ptr, need, stream);
}

extern "C" int spa_gate_bwd_straight_through(const void* x, const void* w, float bias, const float* scores,
                                             const float* s_up, const uint8_t* labels, const void* d_rg,
                                             float loss_scale, const uint8_t* mask, const float* noise,
                                             float temperature, int B, int N, int C, int dtype, float* loss,
                                             void* dx, float* dw, float* db, void* workspace,
                                             size_t workspace_bytes, void* stream) {
  const char* fn = "spa_gate_bwd_straight_through";
  SPA_REQUIRE(mask && d_rg, SPA_ERR_INVALID_ARG, "%s: mask and d_rg are required", fn);
  SPA_REQUIRE(temperature > 0.f && std::isfinite(temperature), SPA_ERR_INVALID_ARG,
              "%s: temperature must be positive and finite, got %g", fn, (double)temperature);
  return gate_bwd_common(fn, x, w, bias, scores, s_up, labels, d_rg, 1, loss_scale,
                         StraightThrough{mask, noise, 1.f / temperature}, B, N, C, dtype, loss, dx, dw, db, workspace,
                         workspace_bytes, stream);
}
