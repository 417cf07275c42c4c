// Blocks that compute the same output tile over different ranges of K meet here, exchange pieces
// through memory and each finish a share of the tile (the many-row residual GEMMs).
//
// The pieces are small and short-lived, so what the exchange costs is what keeping them coherent
// costs.  An agent-scope release writes back an XCD's whole L2 and the acquire invalidates it (5 us a
// launch and more), write-through stores and L2-bypassing loads go to memory and back.  Blocks of ONE XCD
// need neither: they share its L2, to which a block's stores have gone once vmcnt is 0, and a line that the
// block's compute unit has never read is not in its first-level cache.  So the launches put the blocks of
// a tile on one XCD (the dispatcher deals workgroups to the XCDs round-robin), every block tells the
// others which XCD it really runs on, and only if they are not all the same do they fence.  On MI355X
// 256 blocks in groups of four exchange 12 KiB each in 0.4 us more than they take to write them.
//
// Waiting is bounded: a block that has waited too long for the others (they need not be resident at
// the same time) leaves its own share in memory as well, behind a release, says so and goes; the
// block that arrives last finishes the shares of those that have gone.  Every path ends.
//
// Who adds the pieces up does not show in the result: the sum goes over the ranges of K in order.
#pragma once
#include <hip/hip_runtime.h>

#include "ec_internal.h"

namespace ec {

// One group's state, all zero when the launch starts and used by one launch only.
struct MeetSlot {
  unsigned long long arrived;  // low half: per XCD (4 bits each) how many have arrived;
                               // high half: bit z: the block of range z has left its share and gone
  unsigned int fenced;         // how many have made their pieces visible to other XCDs
  unsigned int pad;
};
static_assert(sizeof(MeetSlot) == kMeetSlotBytes, "the workspace and the step prologue count on it");

// arrivals in the low half of MeetSlot::arrived
__device__ __forceinline__ int meet_count(unsigned long long a) {
  const unsigned u = (unsigned)a;
  return (int)((((u & 0x0f0f0f0fu) + ((u >> 4) & 0x0f0f0f0fu)) * 0x01010101u) >> 24);
}

// Called by every thread of block z of Z (at most 4) once the pieces of the OTHER blocks' shares are
// stored.  leave_own() stores the block's own piece of its own share.  Returns the set of shares this
// block finishes (bit per range of K): its own, usually; all pieces of these are readable.
// limit: polls before a block gives up waiting; apart: treat the blocks as if on different XCDs.
template <typename LeaveOwn>
__device__ __forceinline__ unsigned meet_blocks(MeetSlot* slot, int Z, int z, int limit, int apart,
                                                LeaveOwn&& leave_own) {
  __shared__ unsigned verdict;
  constexpr unsigned kGaveUp = 1u << 30, kFence = 1u << 31;
  const unsigned xcc = apart ? (unsigned)z : (__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 7u);  // HW_REG_XCC_ID
  const unsigned long long together = (unsigned long long)((unsigned)Z << (4 * xcc));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned long long one = 1ull << (4 * xcc);
    unsigned long long now = __hip_atomic_fetch_add(&slot->arrived, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + one;
    unsigned v = 1u << z;
    if (meet_count(now) == Z) {
      v |= (unsigned)(now >> 32);   // the last to arrive: for those that have gone, too
    } else {
      for (int n = 0; n < limit && meet_count(now) != Z; ++n) {
        __builtin_amdgcn_s_sleep(1);
        now = __hip_atomic_load(&slot->arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (meet_count(now) != Z) v = kGaveUp;
    else if ((unsigned)now != (unsigned)together) v |= kFence;
    verdict = v;
  }
  __syncthreads();
  unsigned v = verdict;
  if (v & kGaveUp) {
    leave_own();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __hip_atomic_fetch_add(&slot->fenced, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const unsigned long long gone = 1ull << (32 + z);
      const unsigned long long old = __hip_atomic_fetch_add(&slot->arrived, gone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // (if the last one arrived first, it has not seen the mark: this block stays)
      v = meet_count(old) != Z ? 0u : (1u << z) | ((unsigned)old != (unsigned)together ? kFence : 0u);
      verdict = v | kGaveUp;
    }
    __syncthreads();
    v = verdict;
  }
  if (v & kFence) {
    if (threadIdx.x == 0) {
      if (!(v & kGaveUp)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_fetch_add(&slot->fenced, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      // all have arrived, and each comes past one of the two additions without waiting for anyone
      while (__hip_atomic_load(&slot->fenced, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (unsigned)Z)
        __builtin_amdgcn_s_sleep(1);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
  }
  asm volatile("" ::: "memory");
  return __builtin_amdgcn_readfirstlane(v & 0xfu);
}

}  // namespace ec
