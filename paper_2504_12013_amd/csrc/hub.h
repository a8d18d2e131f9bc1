// The hub pass as device code: a kernel of its own (k_hub.hip), or the first workgroups of the pass over
// the other vertices.
#pragma once
#include <algorithm>

#include "chunk.h"
#include "conn.h"
#include "dev_util.h"
#include "entry.h"
#include "hand_over.h"
#include "jet_internal.h"
#include "rec.h"

namespace jet {

constexpr int kHubBlock = 256;
constexpr int kHubWaves = kHubBlock / kWave;
// Workgroups of one hub: one per kHubShare nets (the four of a thread that are in flight together), at most
// kHubShares.
constexpr int kHubShares = 16;
constexpr int kHubShare = 1024;
constexpr int kHubSegment = 508; // nets one lane takes before its nine planes are emptied

// max over 64 lanes of a 64-bit key
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)x, o, kWave);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), o, kWave);
    const unsigned long long y = ((unsigned long long)hi << 32) | lo;
    x = y > x ? y : x;
  }
  return x;
}

struct HubArgs {
  const int32_t *part, *inc, *nw, *sumw, *vw, *hubs;
  const int64_t *voff;
  const uint64_t *ns;
  int32_t nhubs, k;
  unsigned long long *words;  // [kHubGrid / 2 * (k + 1)] sums of shared hubs (hand_over.h), zero between launches
  DevStatus *st;
  const LoopCtl *lc;
  Union u;
  // candidates
  const int32_t *lockstamp;
  const uint8_t *lock_bytes;
  int32_t locked_stamp, tau_q;
  uint64_t *rec;
  uint32_t *inm;
  // rebalancing
  const int32_t *hlist;
  int64_t lmax, dz;
  uint32_t *entries;
};

// The workgroup's share of a hub's nets (incidences q0 + its threads, step threads, ... below q1) into
// row[0..k) and row[k] (benefit), which it clears first.  Every thread calls it; ends with a barrier.
// G: lane group of the weighted form; HW: words of the bit-sliced form (unit net weights).
template <int G, int HW, bool UNIT>
__device__ __forceinline__ void hub_sums(const HubArgs &a, int64_t q0, int64_t q1, int64_t threads, int32_t s,
                                         int32_t *row) {
  const int tid = threadIdx.x, l = lane_id();
  for (int b = tid; b <= a.k; b += kHubBlock) row[b] = 0;
  __syncthreads();
  int32_t ben = 0;
  if (UNIT) {
    constexpr int N = 9, M = 15;  // a wave sums 64 lanes of at most 511
    int32_t total = 0;
    for (int64_t qs = q0; qs < q1; qs += kHubSegment * threads) {  // block-uniform trip count
      uint32_t pl[HW][N] = {}, w[M];
      ben = 0;
      planes_accumulate<HW, N>(a.inc, qs + tid, min(q1, qs + kHubSegment * threads), threads, a.ns, s, pl, ben);
      const int x = planes_combine<kWave, HW, N, M>(pl, w, ben, l);
      total += ben;
      // lane l holds the sums of word x: blocks 32 x + j, spread over the lanes that hold that word
      constexpr int SH = HW == 1 ? 0 : HW == 2 ? 1 : 2;
      for (int j = l >> SH; j < 32; j += kWave >> SH) {
        int32_t c = 0;
#pragma unroll
        for (int p = 0; p < M; ++p) c |= (int32_t)((w[p] >> j) & 1u) << p;
        if (c) atomicAdd(&row[32 * x + j], c);  // blocks of k and above have no pins
      }
    }
    if (l == 0 && total) atomicAdd(&row[a.k], total);
  } else {
    constexpr int NG = kWave / G;
    const int lg = l % G, gi = tid / G;  // group of the workgroup
    int32_t conn[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) conn[b] = 0;
    if (G == 1)
      conn_accumulate_strided<G>(a.inc, q0 + tid, q1, threads, a.nw, a.ns, lg, s, conn, ben);
    else
      conn_accumulate<G>(a.inc, q0 + (int64_t)gi * G, q1, threads, a.nw, a.ns, lg, s, conn, ben);
#pragma unroll
    for (int o = G; o < kWave; o <<= 1) {  // sums over the wave's groups, in every lane
#pragma unroll
      for (int b = 0; b < 8; ++b) conn[b] += __shfl_xor(conn[b], o, kWave);
      ben += __shfl_xor(ben, o, kWave);
    }
#pragma unroll
    for (int b = 0; b < 8; ++b)
      if (b % NG == (l / G) % NG && lg * 8 + b < a.k && conn[b]) atomicAdd(&row[lg * 8 + b], conn[b]);
    if (l == 0 && ben) atomicAdd(&row[a.k], ben);
  }
  __syncthreads();
}

// The work of workgroup bid of nblk on the hubs.  RB: those listed in hlist; otherwise all unlocked hubs.
template <int G, int HW, bool UNIT, bool RB>
__device__ __forceinline__ void hub_work(const HubArgs &a, int32_t bid, int32_t nblk) {
  __shared__ int32_t row[kMaxK + 1];
  __shared__ int32_t s_last;
  const int32_t nh = RB ? a.st->rb_nhub : a.nhubs;
  if (nh == 0) return;
  const int tid = threadIdx.x, l = lane_id(), k = a.k;
  const bool un = a.u.lcs != nullptr;
  int32_t ls0 = a.locked_stamp, tq0 = a.tau_q, unw0 = 0;
  int64_t dz0 = a.dz;
  if (a.lc && !un) {
    ls0 = a.lc->stamp - 1;
    tq0 = a.lc->tau_q;
    dz0 = a.lc->dz;
    unw0 = a.lc->rb_unw;
  }
  const int32_t per = max(1, min(kHubShares, nblk / nh));  // most workgroups of a hub
  unsigned long long scanned = 0ull, examined = 0ull, emitted = 0ull;     // thread 0
  for (int64_t i = bid; i < (int64_t)nh * per; i += nblk) {   // block-uniform trip count
    const int32_t j = (int32_t)(i / per), sub = (int32_t)(i % per);
    const int32_t hi = RB ? a.hlist[j] : j;
    const int32_t v = a.hubs[hi];
    const int32_t s = a.part[v];
    const LoopCtl *h = un ? &a.u.lcs[a.u.vhg[v]] : nullptr;  // the hub's own hypergraph (union)
    if (!RB) {
      const int32_t ls = un ? h->stamp - 1 : ls0;
      const bool off = un && h->phase != kPhJet;
      if (off || (a.lock_bytes ? a.lock_bytes[v] != 0 : a.lockstamp[v] == ls)) {
        if (sub == 0 && tid == 0) a.rec[v] = pack_rec(0, 0xff, s);
        continue;
      }
    }
    const int64_t q0 = a.voff[v], q1 = a.voff[v + 1];
    const int32_t shares =  // uniform
        __builtin_amdgcn_readfirstlane(min(per, (int32_t)(q1 - q0 + kHubShare - 1) / kHubShare));
    if (sub >= shares) continue;  // block-uniform
    hub_sums<G, HW, UNIT>(a, q0 + (int64_t)sub * kHubBlock, q1, (int64_t)shares * kHubBlock, s, row);
    if (shares > 1) {  // so every hub has a workgroup of its own or several: j < kHubGrid / 2
      unsigned long long *words = a.words + (int64_t)j * (k + 1);
      if (tid <= k) {
        const bool last = word_add(&words[tid], row[tid], shares);
        if (tid == k) s_last = last;
      }
      __syncthreads();
      if (!s_last) continue;  // block-uniform
      if (tid <= k && !word_take(&words[tid], shares, &row[tid]))
        if (atomicCAS(&a.st->err, 0, kErrHandOver) == 0) a.st->err_arg = v;
      __syncthreads();
    }
    if (tid < kWave) {
      const int64_t sg0 = un ? (int64_t)a.u.vhg[v] * k : 0;
      const int32_t c = RB && a.vw ? a.vw[v] : 1;
      const int64_t lm = un ? h->lmax : a.lmax, dzz = un ? h->dz : dz0;
      // best target by conn, lowest block on ties: candidates need an adjacent block, a rebalancing move
      // one with room for v outside the deadzone
      unsigned long long key = 0ull;
      for (int b = l; b < k; b += kWave) {
        const int32_t cb = row[b];
        bool ok = b != s && (RB || cb > 0);
        if (RB && ok) {
          const int64_t bwb = a.st->bw[sg0 + b];
          ok = bwb + c <= lm && bwb < dzz;
        }
        const unsigned long long kb =
            ok ? ((unsigned long long)(uint32_t)(cb + 1) << 32) | (uint32_t)(0xffffffffu - (uint32_t)b) : 0ull;
        key = kb > key ? kb : key;
      }
      key = wave_max_u64(key);
      if (tid == 0) {
        const int32_t bestc = (int32_t)(uint32_t)(key >> 32) - 1, bestb = (int32_t)(0xffffffffu - (uint32_t)key);
        const int32_t benefit = row[k];
        scanned += (unsigned long long)(q1 - q0);
        examined += 1ull;
        if (RB) {
          if (bestc >= 0) {
            const int32_t slot = atomicAdd(&a.st->rb_count[sg0 + s], 1);
            write_entry(a.entries + (a.st->rb_off[sg0 + s] + slot) * kEntryWords, true,
                        bestc - (a.sumw[v] - benefit), c, v, bestb, un ? h->rb_unw : unw0);
            emitted += 1ull;
          }
        } else {
          bool cand = false;
          finish_candidate(v, s, bestc > 0 ? bestc : 0, bestb, a.sumw[v], benefit, un ? h->tau_q : tq0, a.rec, &cand);
          if (cand) {
            atomicOr(&a.inm[v >> 5], 1u << (v & 31));
            emitted += 1ull;
          }
        }
      }
    }
    __syncthreads();  // the row is rewritten for the next hub
  }
  if (tid != 0 || examined == 0ull) return;
  if (RB) {
    count_add(a.st, bid, &CtrSlot::rb_inc, (long long)scanned);
    count_add(a.st, bid, &CtrSlot::rb_elig, (long long)examined);
    count_add(a.st, bid, &CtrSlot::rb_ent, (long long)emitted);
  } else {
    count_add(a.st, bid, &CtrSlot::inc_hub, (long long)scanned);
    count_add(a.st, bid, &CtrSlot::n_cand, (long long)emitted);
  }
}

inline HubArgs hub_args(Ctx &c, const int32_t *part, const LoopCtl *lc) {
  HubArgs a{};
  a.part = part;
  a.inc = c.inc;
  a.nw = c.nw;
  a.sumw = c.sumw;
  a.vw = c.vw;
  a.hubs = c.hubs;
  a.voff = c.voff;
  a.ns = c.ns;
  a.nhubs = c.nhubs;
  a.k = c.k;
  a.words = c.hub_words;
  a.st = c.st;
  a.lc = lc;
  a.u = union_of(c);
  a.lockstamp = c.lockstamp;
  a.rec = c.rec;
  a.inm = c.inm;
  a.hlist = c.rb_hlist;
  a.lmax = c.lmax;
  a.entries = c.rb_keys;
  return a;
}

// Workgroups of a pass over the other vertices that take the hubs (a multiple of the eight XCDs, so that the
// others keep theirs).
inline int32_t hub_blocks(const Ctx &c) {
  return (int32_t)(std::min<int64_t>(kHubGrid / 2, (int64_t)c.nhubs * kHubShares) + 7) / 8 * 8;
}
// Both passes of a level as one launch: with unit net weights, where the candidate bits of light vertices
// are ORed into place as the hubs' are.
inline bool hubs_beside_gains(const Ctx &c) { return c.unit_nw && c.nhubs > 0 && c.H == 1; }
inline bool hubs_beside_candidates(const Ctx &c) { return hubs_beside_gains(c) && !light_lanes(c); }

}  // namespace jet
