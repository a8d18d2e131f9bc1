// Sums handed over between workgroups of one launch through single words, with relaxed atomics alone.
// Include after hip/hip_runtime.h.
//
// A word holds the sum of one column in its low half (below 2^31 in all) and the number of workgroups that
// have added to it in its high half.  Nothing has to be ordered between words: whoever takes a word waits until
// all have added to that very word, and each of them adds before it waits for anything, so the wait
// ends.  A release and an acquire fence between the workgroups (a write-back of the L2 and an
// invalidation) cost 3 to 5 us a launch instead.
#pragma once
#include <stdint.h>

namespace jet {

constexpr int32_t kTakeSpins = 1 << 24;  // looks at a word before the wait is given up (never reached)

// Adds to a word; returns whether all the others of `shares` workgroups had added before.
__device__ __forceinline__ bool word_add(unsigned long long *w, int32_t v, int32_t shares) {
  const unsigned long long old = __hip_atomic_fetch_add(w, (1ull << 32) | (unsigned long long)(uint32_t)v,
                                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return (int32_t)(old >> 32) == shares - 1;
}

// The sum of a word to which every one of `shares` workgroups adds; the word is zero again afterwards (for the
// next launch).  False: some workgroup never added.
__device__ __forceinline__ bool word_take(unsigned long long *w, int32_t shares, int32_t *sum) {
  for (int32_t i = 0; i < kTakeSpins; ++i) {
    const unsigned long long x = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((int32_t)(x >> 32) != shares) continue;
    *sum = (int32_t)(uint32_t)x;
    __hip_atomic_store(w, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
  }
  return false;
}

}  // namespace jet
