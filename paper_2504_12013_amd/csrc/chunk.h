// Wave-per-chunk mapping for small nets.  A chunk is a run of consecutive nets with at most 64
// pins in total; one wave holds all of them, one pin per lane, so per-net work needs no atomics
// between waves and no segment search.  Chunk descriptors (first net, number of nets, number of
// pins, first pin) and every pin's net index inside its chunk are built once at set-up, so a lane
// finds its pin and net with one load each.
#pragma once
#include "dev_util.h"

namespace jet {

// Orders this wave's LDS accesses before the following ones (for LDS private to the wave).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace jet
