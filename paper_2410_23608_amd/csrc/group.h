// Launch groups (spa_group_begin / spa_group_end): the calls of the stages of a hierarchy, which are small and do
// not depend on each other except through the gates' score maps, in one launch per step of the path instead of one
// per stage and step.  However small it is, a launch costs the host 3.6 us and the stream 1.6 us (200 dependent
// launches of one workgroup, issued one by one and queued ahead), and a small kernel 2-3 us more of trips to memory.
//
// Between begin and end an entry point only notes its kernel's arguments (thread-local); end launches what was noted
// step by step: gates, packing, attention, attention backward, gate backward, projection backward.  A kernel of a
// group takes the arguments of up to kGroupMax calls, the workgroups of call s being [end[s-1], end[s]).
#pragma once
#include "spa_common.h"

namespace spa {

constexpr int kGroupMax = 4;

template <class A>
struct Members {
  A a[kGroupMax];
  unsigned end[kGroupMax];       // (members past the last: the last one's)
};

// The call a workgroup works for, its number among the call's workgroups and their number.
struct MemberBlock {
  int s;
  unsigned block, blocks;
};
template <class A>
__device__ __forceinline__ MemberBlock member_of(const Members<A>& m, unsigned block) {
  int s = 0;
  while (s < kGroupMax - 1 && block >= m.end[s]) ++s;
  const unsigned from = s > 0 ? m.end[s - 1] : 0u;
  return {s, block - from, m.end[s] - from};
}

// Host side: the noted calls of one kernel.
template <class A>
struct Noted {
  int n = 0;
  A a[kGroupMax];
  unsigned blocks[kGroupMax];
  int add(const char* fn, const A& x, unsigned nblocks) {
    if (n == kGroupMax) return fail(SPA_ERR_UNSUPPORTED, "%s: more than %d calls of a kind in a group", fn, kGroupMax);
    a[n] = x;
    blocks[n++] = nblocks;
    return SPA_OK;
  }
  unsigned members(Members<A>& m) {      // all workgroups; forgets the calls
    unsigned total = 0;
    for (int i = 0; i < kGroupMax; ++i) {
      const int s = i < n ? i : n - 1;
      m.a[i] = a[s];
      if (i < n) total += blocks[i];
      m.end[i] = total;
    }
    n = 0;
    return total;
  }
};

// One per source file that takes part: launch what was noted / forget it.
int group_flush_gates(hipStream_t st);
int group_flush_pack(hipStream_t st);
int group_flush_attention(hipStream_t st);
int group_flush_attention_bwd(hipStream_t st);
int group_flush_gates_bwd(hipStream_t st);
int group_flush_linear(hipStream_t st);
void group_forget_gates();
void group_forget_pack();
void group_forget_attention();
void group_forget_attention_bwd();
void group_forget_linear();

}  // namespace spa
