// Internal helpers shared by the libspa translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "spa.h"

namespace spa {

// ---- host side -------------------------------------------------------------------
int fail(int code, const char* fmt, ...);          // records the message, returns code
int check_launch(const char* what);                // hipGetLastError -> SPA_ERR_HIP

// Launch options (tuning aids and kernel selection for tests), see spa_set_option in spa.h.
struct Options {
  bool fwd_whole, fwd_step64, fwd_plain;   // attn_fwd_short
  bool fwd_tiled;                          // attn_fwd_cfg given
  int fwd_wave_max;                        // attn_fwd_wave_max
  bool bwd_tiled;                          // attn_bwd_short = tiled
  int gemm_tm, gemm_splits, pack_tile;     // 0 = automatic
};
const Options& options();

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool apart(const void* a, size_t na, const void* b, size_t nb) {      // two ranges of memory share no byte
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x + na <= y || y + nb <= x;
}
inline int elem_size(int dtype) { return dtype == SPA_BF16 ? 2 : 4; }

// D_i = <dy_i, out_i> of every (head, packed row) for the attention backward, dy at token positions (attention_bwd.hip)
void launch_dvec(const void* out, const void* dy, const int32_t* gather_idx, const int32_t* cu, int B, int H, int Dh, long lse_stride,
                 float* dvec, hipStream_t st);

extern thread_local bool g_group_open;             // a launch group is open on this thread (group.h)
inline bool group_open() { return g_group_open; }

#define SPA_REQUIRE(cond, code, ...)                 \
  do {                                               \
    if (!(cond)) return ::spa::fail(code, __VA_ARGS__); \
  } while (0)
// For entry points that launch at once whatever the group: nothing of a group is launched when a call of it fails.
#define SPA_REFUSE_IN_GROUP(fn) SPA_REQUIRE(!::spa::group_open(), SPA_ERR_UNSUPPORTED, "%s: cannot be part of a group", fn)

// ---- device side -----------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Number of set bits of a wave-wide ballot below this lane.
__device__ __forceinline__ int rank_in_ballot(uint64_t ballot) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(ballot >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(ballot), 0));
}

// Sum over the wave, in every lane, without LDS (an exchange through it takes 85 cycles, one of these 8 to 16).
template <int CTRL>
__device__ __forceinline__ int add_dpp(int v) { return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false); }
__device__ __forceinline__ int wave_sum(int v) {
  const auto h = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);      // lane ^ 32
  const unsigned a = h[0], b = h[1], c = a + b;
  const auto q = __builtin_amdgcn_permlane16_swap(c, c, false, false);                          // lane ^ 16
  const unsigned d = q[0], e = q[1];
  // rotations by 8 and 4 in a row of 16, quad_perm [2, 3, 0, 1] and [1, 0, 3, 2]
  return add_dpp<0xB1>(add_dpp<0x4E>(add_dpp<0x124>(add_dpp<0x128>((int)(d + e)))));
}

// Inclusive sums over the wave: shifts by 1, 2, 4 and 8 in a row of 16, then the last lane of every other row and of the
// first half to the rows after them.
template <int CTRL, int ROWS>
__device__ __forceinline__ int add_dpp_rows(int v) { return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false); }
__device__ __forceinline__ int wave_scan(int v) {
  v = add_dpp_rows<0x118, 0xF>(add_dpp_rows<0x114, 0xF>(add_dpp_rows<0x112, 0xF>(add_dpp_rows<0x111, 0xF>(v))));
  return add_dpp_rows<0x143, 0xC>(add_dpp_rows<0x142, 0xA>(v));
}
// The value of another lane, without LDS: lane ^ 1, ^ 2 inside a quad, ^ 4 as two shifts.
template <int CTRL, int BANKS = 0xF>
__device__ __forceinline__ float dpp_move(float v, float other = 0.f) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, other), __builtin_bit_cast(int, v), CTRL, 0xF, BANKS, false));
}
template <int MASK>
__device__ __forceinline__ float lane_xor(float v) {
  static_assert(MASK == 1 || MASK == 2 || MASK == 4, "inside a row of 16");
  if (MASK == 1) return dpp_move<0xB1>(v);
  if (MASK == 2) return dpp_move<0x4E>(v);
  return dpp_move<0x114, 0xA>(v, dpp_move<0x104, 0x5>(v));
}
// Sum over G = 4 or 8 adjacent lanes, in every one of them
template <int G>
__device__ __forceinline__ float adjacent_sum(float v) {
  static_assert(G == 4 || G == 8, "a quad or two");
  v += lane_xor<1>(v);
  v += lane_xor<2>(v);
  return G == 8 ? v + lane_xor<4>(v) : v;
}

// 8 bf16 (one 16-byte chunk) <-> 8 floats
__device__ __forceinline__ floatx8 bf16x8_to_float(bf16x8 v) { return __builtin_convertvector(v, floatx8); }
__device__ __forceinline__ bf16x8 float_to_bf16x8(floatx8 v) { return __builtin_convertvector(v, bf16x8); }

__device__ __forceinline__ float sigmoidf_dev(float s) {
  float e = __expf(-fabsf(s));
  float r = 1.0f / (1.0f + e);
  return s >= 0.f ? r : e * r;
}

}  // namespace spa
