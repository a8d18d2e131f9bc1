// Hub vertices (more than kHubDegree incident nets): move candidates (Section 4.1) and rebalancing
// gains (Section 4.3).
//
// Both need conn(v, b) over all incident nets of every hub.  A workgroup takes a hub, or while there
// are fewer hubs than workgroups a share of a long one; then the workgroups of a hub add their sums into
// words (hand_over.h) and the one that completes the last word finishes the hub (best target, record or
// entry), so no second launch waits for the sums.  With unit net weights a lane takes whole nets into
// bit-sliced counts (conn.h), which the wave sums at the end: a net costs a lane a gather and some 15
// instructions.  Eight lanes per net with four exchanges and 24 instructions each bound the passes by
// vector instructions (four cycles each): on levels of 1M row-net vertices candidates took 49 us (now 40)
// and a rebalancing pass 38 us in three launches (25).
#include "hub.h"

namespace jet {

namespace {

// Union: the hubs that may move, by their index in the hub list (one hypergraph: k_rb_list).
__global__ __launch_bounds__(256) void k_rb_hub_list(const int32_t *__restrict__ part, const int32_t *__restrict__ vw,
                                                     const int32_t *__restrict__ hubs, int32_t nhubs, DevStatus *st,
                                                     int32_t *__restrict__ hlist, const LoopCtl *lc, int32_t k,
                                                     Union u) {
  JET_GATE(lc, kPhRb);
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  bool e = false;
  if (i < nhubs) {
    const int32_t v = hubs[i];
    const LoopCtl &h = u.lcs[u.vhg[v]];
    const int64_t bs = st->bw[(int64_t)u.vhg[v] * k + part[v]];
    const int64_t c = vw ? vw[v] : 1;
    e = h.phase == kPhRb && bs > h.lmax && 2 * c <= 3 * (bs - h.A);
  }
  const uint64_t mm = ballot(e);
  if (!mm) return;
  int32_t base = 0;
  if (lane_id() == 0) base = atomicAdd(&st->rb_nhub, __popcll(mm));
  base = __shfl(base, 0, kWave);
  if (e) hlist[base + rank_below(mm)] = i;
}

// candidates
template <int G, int HW, bool UNIT>
__global__ __launch_bounds__(kHubBlock) void k_hub(HubArgs a) {
  JET_GATE(a.lc, kPhJet);
  hub_work<G, HW, UNIT, false>(a, (int32_t)blockIdx.x, (int32_t)gridDim.x);
}

// rebalancing gains
template <int G, int HW, bool UNIT>
__global__ __launch_bounds__(kHubBlock) void k_rb_hub(HubArgs a) {
  JET_GATE(a.lc, kPhRb);
  hub_work<G, HW, UNIT, true>(a, (int32_t)blockIdx.x, (int32_t)gridDim.x);
}

template <bool RB, int G, int HW, bool UNIT>
void hub_launch_form(Ctx &c, int64_t blocks, const HubArgs &a) {
  if constexpr (RB) launch_resident<k_rb_hub<G, HW, UNIT>>(c, blocks, kHubBlock, a);
  else launch_resident<k_hub<G, HW, UNIT>>(c, blocks, kHubBlock, a);
}

template <bool RB>
hipError_t hub_launch(Ctx &c, const HubArgs &a) {
  const int64_t blocks = std::min<int64_t>(kHubGrid, (int64_t)c.nhubs * kHubShares);
#define JET_HUB(G, HW, UNIT) hub_launch_form<RB, G, HW, UNIT>(c, blocks, a)
  if (c.unit_nw) {
    if (c.k <= 32) JET_HUB(1, 1, true);
    else if (c.k <= 64) JET_HUB(1, 2, true);
    else JET_HUB(1, 4, true);
  } else {
    if (c.k <= 8) JET_HUB(1, 1, false);
    else if (c.k <= 16) JET_HUB(2, 1, false);
    else if (c.k <= 32) JET_HUB(4, 1, false);
    else if (c.k <= 64) JET_HUB(8, 1, false);
    else JET_HUB(16, 1, false);
  }
#undef JET_HUB
  return hipGetLastError();
}

}  // namespace

hipError_t launch_candidates_hub(Ctx &c, const int32_t *part, int32_t locked_stamp, const uint8_t *lock_bytes,
                                 int32_t tau_q, const LoopCtl *lc) {
  HubArgs a = hub_args(c, part, lc);
  a.locked_stamp = locked_stamp;
  a.lock_bytes = lock_bytes;
  a.tau_q = tau_q;
  return hub_launch<false>(c, a);
}

hipError_t launch_rb_hubs(Ctx &c, const int32_t *part, int64_t dz, const LoopCtl *lc) {
  if (c.nhubs == 0 || hubs_beside_gains(c)) return hipSuccess;
  if (c.H > 1)
    hipLaunchKernelGGL(k_rb_hub_list, dim3((unsigned)((c.nhubs + 255) / 256)), dim3(256), 0, c.stream, part, c.vw,
                       c.hubs, c.nhubs, c.st, c.rb_hlist, lc, c.k, union_of(c));
  HubArgs a = hub_args(c, part, lc);
  a.dz = dz;
  return hub_launch<true>(c, a);
}

}  // namespace jet
